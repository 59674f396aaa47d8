"""Kernel-level parity: each single-operation entry point against the CPU oracle."""
import numpy as np
import pytest

from oracle import sampling as osamp
from oracle import transformer as otf
from paper_2601_05475_amd import binding, synth

from gpu_common import ATT_REL, check_sampler_on_logits, rel_l2

pytestmark = pytest.mark.gpu


def to_dev(a, dtype):
    """numpy fp32 values -> device tensor of the model dtype; returns (tensor, values as fp32)."""
    import torch
    if dtype == "f32":
        return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda(), np.asarray(a, np.float32)
    t = torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(torch.bfloat16)
    return t.cuda(), t.to(torch.float32).numpy()


def rnd(seed, shape, std=1.0):
    return synth.normal(seed, 9, shape, 0.0, std, "f32")


TOL = {"f32": 2e-5, "bf16": 1e-2}      # relative to the output scale; bf16 outputs are rounded


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_add_rmsnorm(dtype):
    import torch
    rows, d, S = 5, 300, 3
    x = rnd(1, (rows, d)); parts = rnd(2, (S, rows, d), 0.3); g = 1 + rnd(3, (d,), 0.1)
    gd, gv = to_dev(g, dtype)
    xd = torch.from_numpy(x.copy()).cuda(); pd = torch.from_numpy(parts).cuda()
    h = binding.op_add_rmsnorm(xd, pd, gd, 1e-6)
    xs = x.astype(np.float64) + parts.astype(np.float64).sum(0)
    np.testing.assert_allclose(xd.cpu().numpy(), xs, rtol=0, atol=1e-6)
    want = otf.rmsnorm(xs, gv, 1e-6)
    np.testing.assert_allclose(h.float().cpu().numpy(), want, rtol=0, atol=TOL[dtype] * 4)
    h0 = binding.op_add_rmsnorm(xd, None, gd, 1e-6)          # no partials: x untouched
    np.testing.assert_array_equal(h0.float().cpu().numpy(), h.float().cpu().numpy())


@pytest.mark.parametrize("dtype,M,N,K,S", [
    ("f32", 3, 70, 100, 1), ("f32", 3, 70, 100, 3), ("f32", 130, 65, 33, 1),
    ("bf16", 4, 96, 200, 2), ("bf16", 32, 256, 512, 4), ("bf16", 16, 3072, 2048, 1),
    ("bf16", 200, 128, 256, 1), ("bf16", 33, 130, 72, 1),
])
def test_linear(dtype, M, N, K, S):
    a = rnd(4, (M, K)); w = rnd(5, (N, K), 0.05)
    ad, av = to_dev(a, dtype); wd, wv = to_dev(w, dtype)
    print("case: linear", dtype, M, N, K, S, flush=True)
    out = binding.op_linear(ad, wd, S).cpu().numpy().astype(np.float64).sum(0)
    want = otf.linear(av, wv)
    np.testing.assert_allclose(out, want, rtol=0, atol=2e-5 * np.abs(want).max() + 1e-6)


# One output column per wave, up to 32 rows: both row groups, rows past a group, columns past a
# workgroup, K shorter and longer than one pass of the lanes, splits with a short and an empty range.
@pytest.mark.parametrize("dtype,M,N,K,S", [
    ("f32", 1, 5, 4, 1), ("f32", 4, 256, 688, 2), ("f32", 5, 66, 260, 1), ("f32", 9, 7, 1028, 3), ("f32", 32, 130, 512, 4),
    ("bf16", 3, 9, 8, 1), ("bf16", 8, 33, 520, 1), ("bf16", 17, 64, 1032, 2), ("f32", 2, 6, 20, 3),
    # few rows that go to the tiles: many waves with little of K each
    ("f32", 32, 4096, 256, 4), ("bf16", 16, 4100, 264, 4), ("f32", 9, 4096, 1024, 16),
])
def test_linear_few_rows_generic(dtype, M, N, K, S):
    test_linear(dtype, M, N, K, S)
    if S == 1:
        test_linear_swiglu(dtype, M, N, K)


@pytest.mark.parametrize("dtype,M,N,K", [("f32", 5, 70, 100), ("bf16", 4, 96, 200), ("bf16", 32, 512, 256),
                                         ("bf16", 150, 128, 128)])
def test_linear_swiglu(dtype, M, N, K):
    a = rnd(6, (M, K)); wg = rnd(7, (N, K), 0.2); wu = rnd(8, (N, K), 0.2)
    ad, av = to_dev(a, dtype); gd, gv = to_dev(wg, dtype); ud, uv = to_dev(wu, dtype)
    out = binding.op_linear_swiglu(ad, gd, ud).float().cpu().numpy()
    want = otf.silu(otf.linear(av, gv)) * otf.linear(av, uv)
    np.testing.assert_allclose(out, want, rtol=0, atol=TOL[dtype] * np.abs(want).max())


def make_pools(dtype, n_pages, Hkv, pg, hd, seed):
    """Random K / V page pools in the library's page layout; returns device tensors and fp32
    views k[page, kvh, j, :], v[page, kvh, j, :] for the oracle."""
    k = rnd(seed, (n_pages, Hkv, pg, hd)); v = rnd(seed + 1, (n_pages, Hkv, pg, hd))
    kd, kv = to_dev(k, dtype)
    vd, vv = to_dev(v, dtype)
    kp, vp = binding.kv_pages_pack(kd, vd)
    return kp, vp, kv, vv


@pytest.mark.parametrize("dtype,pg", [("f32", 8), ("bf16", 8), ("f32", 32), ("bf16", 64)])
def test_rope_kv_write(dtype, pg):
    import torch
    rows, Hq, Hkv, hd, S, base = 7, 4, 2, 64, 2, 10000.0
    nq = (Hq + 2 * Hkv) * hd
    qkv = rnd(10, (S, rows, nq))
    pos = np.array([0, 1, 5, 130, 4095, 17000, 3], np.int32)
    page = np.array([3, 0, 2, 2, 1, 4, 0], np.int32)
    off = np.array([0, 7, 1, 2, 5, 6, 3], np.int32)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    kp = torch.zeros((5, Hkv, pg * hd), dtype=tdt, device="cuda")
    vp = torch.zeros((5, Hkv, pg * hd), dtype=tdt, device="cuda")
    q = binding.op_rope_kv_write(torch.from_numpy(qkv).cuda(), torch.from_numpy(pos).cuda(),
                                 torch.from_numpy(page).cuda(), torch.from_numpy(off).cuda(),
                                 Hq, Hkv, hd, pg, base, kp, vp)
    full = qkv.astype(np.float64).sum(0).reshape(rows, Hq + 2 * Hkv, hd)
    wq = otf.rope(full[:, :Hq], pos, base)
    wk = otf.rope(full[:, Hq:Hq + Hkv], pos, base)
    wv = full[:, Hq + Hkv:]
    tol = 1e-5 if dtype == "f32" else 2e-2
    np.testing.assert_allclose(q.float().cpu().numpy(), wq, rtol=0, atol=tol)
    ku, vu = binding.kv_pages_unpack(kp, vp, pg, hd)
    kh, vh = ku.float().cpu().numpy(), vu.float().cpu().numpy()
    for r in range(rows):
        np.testing.assert_allclose(kh[page[r], :, off[r], :], wk[r], rtol=0, atol=tol)
        np.testing.assert_allclose(vh[page[r], :, off[r], :], wv[r], rtol=0, atol=tol)
    written = np.zeros((5, pg), bool); written[page, off] = True
    assert np.all(kh[~written[:, None, :, None].repeat(Hkv, 1).repeat(hd, 3)] == 0)


def plant_key(kv, vv, kd_pool, vd_pool, page, kvh, slot, q_row, gain, dtype):
    """Make key `slot` of (page, kvh) a multiple of q_row, so that it takes nearly all of that
    row's softmax weight; host views and device pools are updated alike."""
    import torch
    pg, hd = kv.shape[2], kv.shape[3]
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    kt = torch.from_numpy(np.ascontiguousarray(gain * q_row, np.float32)).to(tdt)
    kv[page, kvh, slot] = kt.to(torch.float32).numpy()
    k_off, _ = binding.kv_page_offsets(pg, hd)
    kd_pool[page, kvh, torch.from_numpy(k_off[slot]).cuda()] = kt.cuda()


def attention_case(dtype, B, Hq, Hkv, hd, pg, P, t, splits=0, seed=20, stride=1, qscale=1.0, plant=()):
    """Decode attention against the oracle.  plant: (b, a, where, pos) tuples: the key at prefix /
    suffix position pos of row (b, a)'s KV head becomes 3 q[b, a] (score ~ 3 sqrt(hd) + the rest
    ~ N(0, 1): that key alone decides the output).  Returns (worst relative L2 over the compared
    rows, out, relative errors of the planted rows)."""
    import torch
    n_pre = -(-P // pg) if P else 0
    per = -(-t // pg) if t else 0
    kpd, vpd, kpv, vpv = make_pools(dtype, max(n_pre, 1), Hkv, pg, hd, seed)
    ksd, vsd, ksv, vsv = make_pools(dtype, max(B * per, 1), Hkv, pg, hd, seed + 2)
    table = np.random.default_rng(seed).permutation(max(B * per, 1)).astype(np.int32).reshape(B, -1) if per else np.zeros((B, 1), np.int32)
    q = rnd(seed + 4, (B, Hq, hd), qscale)
    qd, qv = to_dev(q, dtype)
    G = Hq // Hkv
    for b, a, where, pos in plant:
        if where == "prefix":
            plant_key(kpv, vpv, kpd, vpd, pos // pg, a // G, pos % pg, qv[b, a], 3.0 / qscale, dtype)
        else:
            plant_key(ksv, vsv, ksd, vsd, table[b, pos // pg], a // G, pos % pg, qv[b, a], 3.0 / qscale, dtype)
    print("case: attention", dtype, B, Hq, Hkv, hd, pg, P, t, splits, plant, flush=True)
    out = binding.op_attention_decode(qd, kpd if P else None, vpd if P else None, ksd if t else None,
                                      vsd if t else None, torch.from_numpy(table).cuda() if t else None,
                                      P, t, pg, splits).float().cpu().numpy()

    def want_row(b, a):
        c = a // G
        keys = [kpv[:, c].reshape(-1, hd)[:P]] if P else []
        vals = [vpv[:, c].reshape(-1, hd)[:P]] if P else []
        if t:
            keys.append(ksv[table[b, :per], c].reshape(-1, hd)[:t])
            vals.append(vsv[table[b, :per], c].reshape(-1, hd)[:t])
        return otf.attention_one(qv[b, a], np.concatenate(keys), np.concatenate(vals))

    worst = 0.0
    for b in range(B):
        for a in range(Hq):
            if (b * Hq + a) % stride:
                continue
            worst = max(worst, rel_l2(out[b, a], want_row(b, a)))
    planted = [rel_l2(out[b, a], want_row(b, a)) for b, a, _, _ in plant]
    return worst, out, planted


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,Hq,Hkv,hd,pg,P,t", [
    (4, 4, 2, 64, 4, 128, 16), (3, 8, 2, 128, 64, 300, 70), (2, 4, 4, 32, 8, 0, 9),
    (5, 6, 2, 64, 16, 77, 0), (1, 4, 1, 128, 64, 1, 1), (32, 32, 8, 128, 64, 1024, 130),
])
def test_attention_decode(dtype, B, Hq, Hkv, hd, pg, P, t):
    worst, _, _ = attention_case(dtype, B, Hq, Hkv, hd, pg, P, t)
    assert worst < ATT_REL[dtype], worst


# The generic kernel's quads of keys and coordinates: head_dim or page sizes that do not allow them, the
# largest head_dim, a prefix and suffixes that end inside a quad, more blocks than waves and fewer.
@pytest.mark.parametrize("dtype,B,Hq,Hkv,hd,pg,P,t", [
    ("f32", 2, 4, 2, 6, 8, 21, 3), ("f32", 3, 2, 1, 64, 2, 9, 5), ("bf16", 2, 4, 2, 64, 1, 7, 2), ("f32", 1, 2, 1, 256, 4, 130, 70),
    ("bf16", 2, 6, 2, 20, 8, 66, 65), ("f32", 2, 4, 4, 64, 4, 700, 63), ("bf16", 1, 4, 2, 256, 32, 65, 1),
])
def test_attention_decode_generic_quads(dtype, B, Hq, Hkv, hd, pg, P, t):
    worst, _, _ = attention_case(dtype, B, Hq, Hkv, hd, pg, P, t)
    assert worst < ATT_REL[dtype], worst


@pytest.mark.parametrize("dtype,B,Hq,Hkv,hd,pg,P,t,splits", [
    ("f32", 5, 4, 2, 64, 4, 30, 19, 0), ("bf16", 3, 8, 2, 96, 64, 100, 70, 0),                             # the generic kernel
    ("bf16", 6, 8, 2, 128, 64, 300, 200, 0), ("bf16", 4, 8, 4, 64, 64, 0, 130, 0),                          # a workgroup per candidate and KV head
    ("bf16", 9, 32, 8, 128, 64, 1000, 333, 0), ("bf16", 6, 8, 2, 128, 64, 300, 200, 2), ("bf16", 4, 8, 4, 64, 64, 0, 130, 1),   # split keys
    ("bf16", 64, 8, 2, 128, 64, 400, 130, 3),                                                               # ... four row blocks per prefix item
])
def test_attention_decode_candidates_of_different_lengths(dtype, B, Hq, Hkv, hd, pg, P, t, splits):
    """row_len: every candidate attends to its own number of suffix keys (1 .. t; some end inside
    the first block, some on a block or page edge, one is at the maximum), against the oracle's
    attention on exactly those keys."""
    import torch
    n_pre = -(-P // pg) if P else 0
    per = -(-t // pg)
    kpd, vpd, kpv, vpv = make_pools(dtype, max(n_pre, 1), Hkv, pg, hd, 41)
    ksd, vsd, ksv, vsv = make_pools(dtype, B * per, Hkv, pg, hd, 43)
    rng = np.random.default_rng(44)
    table = rng.permutation(B * per).astype(np.int32).reshape(B, per)
    lens = rng.integers(1, t + 1, B).astype(np.int32)
    lens[0], lens[1] = t, 1
    if B > 2:
        lens[2] = min(t, 32)
    if B > 3:
        lens[3] = min(t, pg)
    q = rnd(45, (B, Hq, hd))
    qd, qv = to_dev(q, dtype)
    print("case: ragged attention", dtype, B, Hq, Hkv, hd, pg, P, t, lens.tolist(), flush=True)
    out = binding.op_attention_decode(qd, kpd if P else None, vpd if P else None, ksd, vsd,
                                      torch.from_numpy(table).cuda(), P, t, pg, splits,
                                      row_len=torch.from_numpy(lens).cuda()).float().cpu().numpy()
    G = Hq // Hkv
    worst = 0.0
    for b in range(B):
        for a in range(Hq):
            c = a // G
            keys = [kpv[:, c].reshape(-1, hd)[:P]] if P else []
            vals = [vpv[:, c].reshape(-1, hd)[:P]] if P else []
            keys.append(ksv[table[b], c].reshape(-1, hd)[:lens[b]])
            vals.append(vsv[table[b], c].reshape(-1, hd)[:lens[b]])
            want = otf.attention_one(qv[b, a], np.concatenate(keys), np.concatenate(vals))
            worst = max(worst, rel_l2(out[b, a], want))
    assert worst < ATT_REL[dtype], worst


@pytest.mark.parametrize("B,Hq,Hkv,hd,P,t,stride", [
    (32, 32, 8, 128, 4096, 512, 7),      # 8B-shape headline workload at its last step
    (32, 32, 8, 128, 4096, 1, 7),        # ... and at its first
    (16, 32, 8, 64, 2048, 256, 5),       # 1B shape
    (64, 40, 8, 128, 16384, 1024, 41),   # 32B shape: 320 query rows per KV head, 3 row blocks
    (64, 32, 8, 128, 4096, 0, 13),       # reranking fan-out, prefix only
    (2, 8, 8, 128, 63, 65, 1), (3, 8, 4, 64, 65, 64, 1), (5, 16, 2, 128, 129, 127, 1),
    (1, 32, 1, 64, 128, 129, 1), (7, 4, 2, 128, 0, 200, 1), (33, 8, 2, 128, 257, 1, 1),
    # many query rows per KV head
    (50, 32, 8, 128, 1000, 70, 3),       # 7 row blocks (the last of 8 rows), last page of 40 keys
    # (these two by a workgroup per candidate and KV head; test_attention_decode_short_contexts asks for their split form)
    (64, 32, 2, 64, 200, 33, 17),        # head_dim 64, 32 row blocks, last page of 8 keys
    (48, 16, 4, 128, 130, 5, 1),         # 6 row blocks, 3 pages (the last with 2 keys)
    (64, 32, 8, 128, 100, 0, 3),         # 8 row blocks, one key split, no suffix: every item writes its outputs itself
    (72, 32, 8, 128, 700, 40, 5),        # 9 row blocks: three items of 4, 4 and 1 row blocks per KV head and split
])
def test_attention_decode_mfma_shapes(B, Hq, Hkv, hd, P, t, stride):
    worst, _, _ = attention_case("bf16", B, Hq, Hkv, hd, 64, P, t, stride=stride)
    assert worst < ATT_REL["bf16"], worst


@pytest.mark.parametrize("B,Hq,Hkv,hd,P,t,splits", [
    # one workgroup per candidate and KV head: its most blocks at each head_dim and workgroup count and the first past them, fewer blocks
    # than waves, 32 query heads per KV head, one, no prefix, no suffix
    (2, 8, 2, 64, 1248, 32, 0), (2, 8, 2, 64, 1249, 32, 0), (3, 8, 2, 128, 513, 193, 0), (3, 8, 2, 128, 545, 193, 0), (33, 8, 8, 64, 417, 40, 0),
    (33, 8, 8, 64, 449, 40, 0), (64, 8, 8, 128, 64, 40, 0), (64, 8, 8, 128, 65, 40, 0), (3, 8, 8, 128, 128, 0, 0), (3, 8, 8, 128, 129, 0, 0),
    (3, 8, 8, 128, 512, 0, 0), (3, 8, 8, 128, 513, 0, 0), (2, 32, 1, 128, 95, 33, 0), (3, 2, 2, 64, 1, 1, 0), (5, 4, 2, 128, 0, 65, 0), (6, 8, 4, 64, 257, 0, 0),
    (65, 8, 8, 64, 70, 40, 0),             # 520 workgroups: split
    # blocks that were past the first edges of that form
    (2, 8, 2, 64, 1504, 32, 0), (2, 8, 2, 64, 1505, 32, 0), (3, 8, 2, 128, 801, 193, 0), (3, 8, 2, 128, 833, 193, 0), (64, 8, 8, 128, 641, 250, 0),
    (64, 8, 8, 128, 673, 250, 0),
    # the split form at sizes that no longer take it by themselves
    (64, 32, 8, 128, 100, 0, 1), (72, 32, 8, 128, 700, 40, 1), (2, 8, 8, 128, 63, 65, 1), (3, 8, 4, 64, 65, 64, 2), (48, 16, 4, 128, 130, 5, 1),
    (7, 4, 2, 128, 0, 200, 1), (1, 32, 1, 64, 128, 129, 1), (4, 6, 2, 64, 250, 70, 2), (64, 32, 2, 64, 200, 33, 2)])
def test_attention_decode_short_contexts(B, Hq, Hkv, hd, P, t, splits):
    plant = [(B - 1, Hq - 1, "prefix", P - 1)] if P > 1 else []
    if t > 1:
        plant.append((B // 2, 0, "suffix", t - 1))
    worst, _, planted = attention_case("bf16", B, Hq, Hkv, hd, 64, P, t, stride=max(1, B * Hq // 150), splits=splits, plant=plant)
    assert max(planted, default=0.0) < ATT_REL["bf16"] and worst < ATT_REL["bf16"], (worst, planted)


@pytest.mark.parametrize("B,Hq,Hkv,hd,P,t", [
    (64, 32, 8, 128, 640, 250), (33, 8, 8, 128, 300, 40), (33, 8, 8, 128, 96, 40), (16, 32, 32, 64, 1472, 64), (64, 8, 8, 64, 500, 33),
    (64, 32, 8, 64, 1504, 1), (4, 8, 8, 128, 700, 100), (2, 8, 8, 64, 1280, 33), (64, 8, 8, 128, 0, 64), (40, 8, 8, 64, 0, 300), (40, 8, 8, 64, 300, 0),
    (3, 8, 8, 128, 200, 0), (3, 8, 8, 128, 512, 0)])
def test_attention_decode_keeps_the_split_form_where_it_is_faster(B, Hq, Hkv, hd, P, t):
    """Contexts past those of one workgroup per candidate and KV head, two rounds of such workgroups, prefixes or suffixes alone: the
    bits of the split form, which a split count asks for."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(17 * P + t)
    normal = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)  # noqa: E731
    per = max(1, -(-t // 64))
    q, k, v = normal(B, Hq, hd), normal(max(1, -(-P // 64)), Hkv, 64 * hd), normal(max(1, -(-P // 64)), Hkv, 64 * hd)
    ks, vs = normal(B * per, Hkv, 64 * hd), normal(B * per, Hkv, 64 * hd)
    table = torch.randperm(B * per, generator=g, device="cuda").to(torch.int32).reshape(B, per)
    splits = max(1, binding.op_attention_decode_plan(B, Hq, Hkv, hd, 64, P, t, 0)["splits"])
    print("case: split form", B, Hq, Hkv, hd, P, t, splits, flush=True)
    got = [binding.op_attention_decode(q, k, v, ks, vs, table, P, t, 64, prefix_splits=n) for n in (0, splits)]
    assert not got[0].isnan().any() and torch.equal(got[0], got[1])


@pytest.mark.parametrize("Hq,hd,B,P", [(8, 128, 57, 20), (8, 64, 57, 33), (8, 128, 57, 96), (8, 64, 72, 127), (8, 128, 72, 160),
                                       (10, 128, 64, 415)])
def test_attention_decode_ring(Hq, hd, B, P):
    """Many query rows, blocks through the ring of LDS stages: ranges shorter than the ring (1 to 3
    blocks), one round and more (4, 5, 13 blocks, in one split), a last block that is partly
    empty, row blocks of four rows and waves without any."""
    worst, _, _ = attention_case("bf16", B, Hq, 2, hd, 64, P, 3, splits=1)
    assert worst < ATT_REL["bf16"], worst


@pytest.mark.parametrize("B,Hq,Hkv,hd,P,t,plant", [
    # 8B headline shape at its last step: one key deep inside the last prefix split, one in the
    # last 32-key block of a candidate's last suffix page, one in a middle page
    (32, 32, 8, 128, 4096, 512, [(5, 9, "prefix", 4000), (31, 31, "suffix", 500), (17, 2, "suffix", 200), (0, 0, "prefix", 33)]),
    # 32B shape: 320 query rows per KV head, 128 blocks per... many prefix splits
    (64, 40, 8, 128, 16384, 1024, [(63, 39, "prefix", 16383), (40, 17, "prefix", 9000), (7, 3, "suffix", 1023), (22, 36, "suffix", 70)]),
    (16, 32, 8, 64, 2048, 256, [(15, 31, "prefix", 2047), (3, 4, "suffix", 255), (9, 20, "suffix", 64)]),       # 1B shape
    (64, 32, 8, 128, 4096, 0, [(63, 0, "prefix", 4095), (1, 30, "prefix", 2049)]),                                # prefix only
    (7, 4, 2, 128, 0, 200, [(6, 3, "suffix", 199), (0, 0, "suffix", 130)]),                                       # suffix only
])
def test_attention_decode_one_key_decides(B, Hq, Hkv, hd, P, t, plant):
    """A key far inside a late prefix split or a late suffix page carries nearly all the weight of
    one row: a kernel that dropped its block, its page or its split's partial state would be O(1)
    wrong there."""
    worst, _, planted = attention_case("bf16", B, Hq, Hkv, hd, 64, P, t, stride=37, plant=plant)
    assert max(planted) < ATT_REL["bf16"], planted
    assert worst < ATT_REL["bf16"], worst


def test_attention_split_count_invariance():
    plant = [(7, 31, "prefix", 2040), (2, 5, "prefix", 1000)]
    outs = [attention_case("bf16", 8, 32, 8, 128, 64, 2048, 100, splits=s, plant=plant) for s in (1, 2, 8, 32)]
    for worst, o, planted in outs:
        assert worst < ATT_REL["bf16"] and max(planted) < ATT_REL["bf16"], (worst, planted)
    for _, o, _ in outs[1:]:
        # different splits round differently, in the last bf16 bit of the output at most
        rel = np.linalg.norm(o - outs[0][1], axis=-1) / np.linalg.norm(outs[0][1], axis=-1)
        assert rel.max() < 6e-3, rel.max()


def test_attention_split_count_invariance_many_rows():
    """The same with 256 query rows per KV head (8 row blocks) and a ragged last page."""
    outs = [attention_case("bf16", 64, 32, 8, 128, 64, 2048 + 40, 3, splits=s, stride=29) for s in (1, 2, 8, 16)]
    for worst, o, _ in outs:
        assert worst < ATT_REL["bf16"], worst
    for _, o, _ in outs[1:]:
        rel = np.linalg.norm(o - outs[0][1], axis=-1) / np.linalg.norm(outs[0][1], axis=-1)
        assert rel.max() < 6e-3, rel.max()


def test_stream_handle_is_the_current_stream():
    import torch
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(torch.cuda.Stream()):
        assert binding._stream() == torch.cuda.current_stream().cuda_stream != 0
    assert binding._stream() == torch.cuda.current_stream().cuda_stream


def test_kernels_are_run_to_run_identical():
    """Every MFMA kernel twice on the same inputs: bit-identical outputs.  (A vector instruction
    that reads matrix-core results before they have landed shows up here as last-bit noise long
    before it shows up in a tolerance.)"""
    import torch

    def twice(name, f):
        a = f(); torch.cuda.synchronize(); b = f(); torch.cuda.synchronize()
        assert torch.equal(a, b), name

    for M, N, K in [(1, 32000, 2048), (40, 3072, 2048), (32, 4096, 14336)]:
        a = binding.op_pack_tiled(to_dev(rnd(190, (M, K)), "bf16")[0])
        w = binding.op_pack_tiled(to_dev(rnd(191, (N, K), 0.05), "bf16")[0])
        w2 = binding.op_pack_tiled(to_dev(rnd(192, (N, K), 0.05), "bf16")[0])
        S = binding.op_linear_splits("bf16", M, N, K, True)
        twice(f"few-row linear {M} {N} {K}", lambda: binding.op_linear(a, w, S, tiled_shape=(M, N, K)))
        twice(f"few-row swiglu {M} {N} {K}", lambda: binding.op_linear_swiglu(a, w, w2, tiled_shape=(M, N, K)))
    for M, N, K in [(232, 2048, 2048), (3000, 4096, 512)]:
        a = binding.op_pack_tiled(to_dev(rnd(193, (M, K)), "bf16")[0])
        w = binding.op_pack_tiled(to_dev(rnd(194, (N, K), 0.05), "bf16")[0])
        twice(f"gemm {M} {N} {K}", lambda: binding.op_linear(a, w, 1, tiled_shape=(M, N, K)))
    pg = 64
    for Hq, Hkv, hd, P, rows, pos0 in [(32, 8, 64, 40, 40, 0), (32, 8, 128, 1024, 64, 960), (8, 2, 128, 330, 200, 130)]:
        npg = -(-P // pg)
        kp = to_dev(rnd(195, (npg, Hkv, pg * hd)), "bf16")[0]; vp = to_dev(rnd(196, (npg, Hkv, pg * hd)), "bf16")[0]
        q = to_dev(rnd(197, (rows, Hq, hd)), "bf16")[0]
        items = torch.tensor([[j, min(64, rows - j), pos0 + j, -1] for j in range(0, rows, 64)], dtype=torch.int32, device="cuda")
        twice(f"prefill attention {Hq} {Hkv} {hd} {P} {rows}",
              lambda: binding.op_attention_prefill(q, items, kp, vp, None, None, None, P, pg, False))
    for B, Hq, Hkv, hd, P, t in [(16, 32, 8, 64, 1000, 3), (32, 32, 8, 128, 4096, 200), (64, 40, 8, 128, 2048, 70)]:
        per = -(-t // pg)
        kp = to_dev(rnd(198, (-(-P // pg), Hkv, pg * hd)), "bf16")[0]; vp = to_dev(rnd(199, (-(-P // pg), Hkv, pg * hd)), "bf16")[0]
        ks = to_dev(rnd(200, (B * per, Hkv, pg * hd)), "bf16")[0]; vs = to_dev(rnd(201, (B * per, Hkv, pg * hd)), "bf16")[0]
        table = torch.arange(B * per, dtype=torch.int32, device="cuda").reshape(B, per)
        q = to_dev(rnd(202, (B, Hq, hd)), "bf16")[0]
        twice(f"decode attention {B} {Hq} {Hkv} {hd} {P} {t}",
              lambda: binding.op_attention_decode(q, kp, vp, ks, vs, table, P, t, pg))


def test_sample_op_cases():
    import torch
    V, B = 128256, 32
    lg = rnd(30, (B, V), 1.28)
    us = synth.uniforms(31, 1, (B,))
    ld, ud = torch.from_numpy(lg).cuda(), torch.from_numpy(us).cuda()
    toks, topk = binding.op_sample(ld, 0.7, 50, ud, want_topk=True)
    toks, topk = toks.cpu().numpy(), topk.cpu().numpy()
    ok = sum(check_sampler_on_logits(lg[b], 0.7, 50, us[b], toks[b], topk[b]) for b in range(B))
    assert ok >= B - 1
    # shared row: every candidate reads row 0
    t2 = binding.op_sample(ld, 0.7, 50, ud, shared_row=True).cpu().numpy()
    for b in range(B):
        check_sampler_on_logits(lg[0], 0.7, 50, us[b], t2[b])
    # all logits equal: the floor(u k)-th lowest id; k not a power of two; ties cut by id
    eq = torch.zeros((4, 4096), device="cuda")
    u4 = torch.tensor([0.0, 0.26, 0.5, 0.99], device="cuda")
    t3, k3 = binding.op_sample(eq, 0.7, 10, u4, want_topk=True)
    assert t3.cpu().tolist() == [0, 2, 5, 9] and k3.cpu().numpy().tolist() == [list(range(10))] * 4
    # duplicates straddling the cut, negative values, -0.0 vs +0.0
    row = np.array([1.0, -0.0, 0.0, 1.0, -3.0, 0.0, 1.0, 2.0] + [-9.0] * 56, np.float32)
    t4, k4 = binding.op_sample(torch.from_numpy(row[None]).cuda(), 1.0, 5, torch.tensor([0.999], device="cuda"), want_topk=True)
    assert k4.cpu().numpy().tolist() == [[7, 0, 3, 6, 1]]
    assert check_sampler_on_logits(row, 1.0, 5, 0.999, int(t4.cpu()[0]))
    # argmax, lowest id on ties
    g = binding.op_sample(torch.from_numpy(row[None]).cuda(), 0.0, 5, torch.tensor([0.5], device="cuda"))
    assert int(g.cpu()[0]) == 7
    g = binding.op_sample(eq, 1.0, 1, u4)
    assert g.cpu().tolist() == [0, 0, 0, 0]
    # u just below 1 -> last entry; tiny vocab below k
    small = torch.from_numpy(rnd(32, (2, 7))).cuda()
    t5, k5 = binding.op_sample(small, 0.9, 50, torch.tensor([1 - 2 ** -24, 0.0], device="cuda"), want_topk=True)
    assert k5.shape == (2, 7) and int(t5.cpu()[0]) == int(k5.cpu()[0, -1]) and int(t5.cpu()[1]) == int(k5.cpu()[1, 0])


@pytest.mark.parametrize("V,k,T,scale", [
    (128256, 1, 0.7, 1.28),        # k = 1 with T > 0: argmax path
    (128256, 2, 0.6, 1.28), (128256, 50, 0.6, 1.28), (128256, 64, 1.0, 0.01), (128256, 65, 0.7, 30.0),
    (128256, 400, 0.7, 1.28),      # 512 thread groups: the candidate list is near its capacity
    (128256, 1000, 0.7, 1.28),     # the list overflows: radix selection
    (128256, 4096, 1.3, 1.28),     # k above the fast path
    (4096, 50, 0.7, 1.0), (4100, 50, 0.7, 1.0), (4095, 50, 0.7, 1.0), (1000, 200, 0.7, 1.0),
])
def test_sample_selection_paths(V, k, T, scale):
    """Top-k ids bit-exact on both selection paths (threshold selection and radix selection),
    including rows quantised to few distinct values (many ties at the cut)."""
    import torch
    B = 3
    lg = rnd(33 + k, (B, V), scale)
    lg[1] = np.round(lg[1] * 4) / 4 if scale >= 1 else np.round(lg[1] * 400) / 400     # heavy ties
    lg[2, : V // 2] = lg[2, V // 2: 2 * (V // 2)]                                         # every value twice
    us = synth.uniforms(34, 1, (B,))
    print("case: sample paths", V, k, T, scale, flush=True)
    toks, topk = binding.op_sample(torch.from_numpy(lg).cuda(), T, k, torch.from_numpy(us).cuda(), want_topk=True)
    toks, topk = toks.cpu().numpy(), topk.cpu().numpy()
    for b in range(B):
        check_sampler_on_logits(lg[b], T, k, us[b], toks[b], topk[b])


@pytest.mark.parametrize("V,k", [(4096, 2), (4096, 224), (4099, 50), (32768, 50), (32768, 225), (32772, 64), (32771, 128),
                                 (65536, 224)])
def test_sample_group_selection(V, k):
    """The one-pass selection at the edges of its rule (k = 224, rows of 32768 values in registers,
    rows not a multiple of 16 bytes): a random row, rows that rise and fall (the largest
    values lie in a few thread groups, so the candidate list is sixteen times k or overflows), a
    row with fewer values than k above -inf, and a row of twelve distinct values.  Ids bit-exact."""
    import torch
    T = 0.7
    lg = rnd(530 + k, (5, V), 1.28)
    ramp = np.arange(V, dtype=np.float32) * np.float32(1e-4)
    lg[1], lg[2] = ramp, -ramp
    lg[3] = -np.inf
    lg[3, 7: 7 + (k + 1) // 2] = rnd(531, ((k + 1) // 2,), 1.0)
    lg[4] = np.round(lg[4] * 1.5) / 1.5
    us = synth.uniforms(532, 1, (5,))
    print("case: sample groups", V, k, flush=True)
    toks, topk = binding.op_sample(torch.from_numpy(lg).cuda(), T, k, torch.from_numpy(us).cuda(), want_topk=True)
    toks, topk = toks.cpu().numpy(), topk.cpu().numpy()
    for b in range(5):
        check_sampler_on_logits(lg[b], T, k, us[b], toks[b], topk[b])


@pytest.mark.parametrize("k,c", [(2, 385), (50, 384), (50, 385), (50, 1024), (200, 1500), (224, 385), (224, 4096)])
def test_sample_clustered_rows(k, c):
    """The candidate list cut down a second time: c large values side by side in falling, rising and random
    order, and in two values only (more ties than the cut can part).  Ids bit-exact."""
    import torch
    V, T = 32000, 0.7
    lg = np.full((5, V), -50.0, np.float32) + rnd(540, (5, V), 0.1)
    big = np.linspace(1.0, 4.0, c, dtype=np.float32)
    for b, x in enumerate((big, big[::-1], np.random.default_rng(k + c).permutation(big), np.where(np.arange(c) % 3 == 0, 2.0, 1.5))):
        at = 4096 * b + 8
        lg[b, at: at + c] = x
    lg[4, 17: 17 + 6 * c: 6] = big                      # spread out: every sixth place
    us = synth.uniforms(541, 1, (5,))
    print("case: sample clustered", k, c, flush=True)
    toks, topk = binding.op_sample(torch.from_numpy(lg).cuda(), T, k, torch.from_numpy(us).cuda(), want_topk=True)
    toks, topk = toks.cpu().numpy(), topk.cpu().numpy()
    for b in range(5):
        check_sampler_on_logits(lg[b], T, k, us[b], toks[b], topk[b])


def _top4_per_group(row):
    """Reference for the LM head's lists: ids of the four largest of every 64 consecutive logits
    under (value descending, id ascending)."""
    g = row.reshape(-1, 64).astype(np.float64)
    order = np.lexsort((np.broadcast_to(np.arange(64), g.shape), -g), axis=1)[:, :4]
    return order + 64 * np.arange(g.shape[0])[:, None]


@pytest.mark.parametrize("M,N,K", [(32, 65536, 256), (5, 131072, 512), (1, 65664, 256)])
def test_lm_head_top_lists(M, N, K):
    """The LM head's logits against the oracle's linear layer, and its per-group top lists against
    a plain selection on the device's own logits (ids and values bit-exact, ties by lower id:
    the weights are coarse so that equal logits are common)."""
    a = rnd(270, (M, K)); w = np.round(rnd(271, (N, K), 0.05) * 64) / 64
    ad, av = to_dev(a, "bf16"); wd, wv = to_dev(w, "bf16")
    if M == 5:                                     # rows of few distinct values: many ties inside a group
        av = np.sign(av); ad, av = to_dev(av, "bf16")
    print("case: lm head lists", M, N, K, flush=True)
    logits, lists = binding.op_lm_head(binding.op_pack_tiled(ad), binding.op_pack_tiled(wd), (M, N, K))
    logits, lists = logits.cpu().numpy(), lists.cpu().numpy()
    want = otf.linear(av, wv)
    np.testing.assert_allclose(logits, want, rtol=0, atol=2e-5 * np.abs(want).max() + 1e-6)
    for m in range(M):
        ids = _top4_per_group(logits[m])
        np.testing.assert_array_equal(lists[m, :, :, 1], ids)
        np.testing.assert_array_equal(lists[m, :, :, 0].view(np.float32) + 0.0, logits[m][ids] + 0.0)


def test_sample_with_top_lists():
    """Sampling from the LM head's lists instead of whole rows, on rows built to order (one-hot
    activations, so a row of logits is a row of bf16 weights, exactly): random rows at three
    scales (bf16 values tie often), a row whose largest values all sit in one group of 64 (the lists
    are inconclusive and the kernel must select from the whole row), a row of equal values, a row
    where exactly four of the top k share a group.  Ids and top-k lists equal the oracle sampler's
    on the device's logits for every temperature / k pair, with and without the lists in use."""
    import torch
    V, K, B = 65536, 256, 8
    rng = np.random.default_rng(272)
    rows = np.zeros((B, V), np.float32)
    rows[0] = rng.standard_normal(V) * 1.28
    rows[1] = rng.standard_normal(V) * 8.0
    rows[2] = rng.standard_normal(V) * 0.05
    rows[3] = rng.standard_normal(V); rows[3, 64 * 5: 64 * 5 + 40] += 9.0          # 40 of the top 50 in group 5
    rows[4] = 0.5                                                                    # all equal
    rows[5] = rng.standard_normal(V); rows[5, [700, 701, 702, 703]] = [9.0, 8.5, 8.0, 7.5]   # four of one group on top
    rows[6] = np.round(rng.standard_normal(V) * 2) / 2                               # few distinct values
    rows[7] = rng.standard_normal(V); rows[7, 64 * 900 + 3] = 30.0                   # one dominant id
    rows_d, rows_v = to_dev(rows, "bf16")
    a = np.zeros((B, K), np.float32); a[np.arange(B), np.arange(B)] = 1.0
    w = np.zeros((V, K), np.float32); w[:, :B] = rows_v.T
    ad, _ = to_dev(a, "bf16"); wd, _ = to_dev(w, "bf16")
    logits, lists = binding.op_lm_head(binding.op_pack_tiled(ad), binding.op_pack_tiled(wd), (B, V, K))
    lg = logits.cpu().numpy()
    np.testing.assert_array_equal(lg, rows_v)
    us = synth.uniforms(273, 1, (B,))
    ud = torch.from_numpy(us).cuda()
    for T, k in [(0.7, 50), (1.0, 64), (0.7, 65), (0.3, 2), (1.3, 5), (0.0, 50), (0.7, 1)]:
        print("case: sample lists", T, k, flush=True)
        toks, topk = binding.op_sample_lists(logits, lists, T, k, ud, want_topk=True)
        toks, topk = toks.cpu().numpy(), topk.cpu().numpy()
        for b in range(B):
            check_sampler_on_logits(lg[b], T, k, us[b], toks[b], topk[b])
        # the same ids as the whole-row sampler
        t2, k2 = binding.op_sample(logits, T, k, ud, want_topk=True)
        np.testing.assert_array_equal(topk, k2.cpu().numpy())
        np.testing.assert_array_equal(toks, t2.cpu().numpy())
    # every candidate reading row 0 of both
    t3 = binding.op_sample_lists(logits, lists, 0.7, 50, ud, shared_row=True).cpu().numpy()
    for b in range(B):
        check_sampler_on_logits(lg[0], 0.7, 50, us[b], t3[b])


def test_reward_score_op():
    import torch
    V, B, R = 128256, 64, 8
    lg = rnd(40, (B, V), 1.28)
    ids = synth.reward_token_ids(synth.WORKLOADS["8b-rerank"], R)
    vals = np.arange(R, dtype=np.float32)
    lp, sc, rk = binding.op_reward_score(torch.from_numpy(lg).cuda(), torch.from_numpy(ids).cuda(),
                                         torch.from_numpy(vals).cuda(), 0.7)
    lp, sc, rk = lp.cpu().numpy(), sc.cpu().numpy(), rk.cpu().numpy()
    want_lp = np.stack([osamp.reward_logprobs(lg[b], ids) for b in range(B)])
    np.testing.assert_allclose(lp, want_lp, rtol=0, atol=2e-5)
    want_sc = np.array([osamp.expected_value(want_lp[b], vals, 0.7) for b in range(B)])
    np.testing.assert_allclose(sc, want_sc, rtol=0, atol=2e-5)
    assert list(rk) == list(osamp.rank(sc))
    # equal reward logits with labels 0..4 -> exactly 2; ties ranked by index
    flat = np.zeros((3, 100), np.float32); flat[1, 50] = 5.0
    lp, sc, rk = binding.op_reward_score(torch.from_numpy(flat).cuda(), torch.arange(5, dtype=torch.int32, device="cuda"),
                                         torch.arange(5, dtype=torch.float32, device="cuda"), 1.0)
    assert sc.cpu().tolist() == [2.0, 2.0, 2.0] and rk.cpu().tolist() == [0, 1, 2]


# ---------------------------------------------------------------- tiled bf16 MFMA kernels
def test_pack_tiled_roundtrip():
    import torch
    for rows, K in [(32, 64), (33, 128), (100, 256), (4096, 512)]:
        t = torch.from_numpy(rnd(50, (rows, K))).to(torch.bfloat16).cuda()
        flat = binding.op_pack_tiled(t)
        assert flat.numel() == ((rows + 31) // 32 * 32) * K
        back = binding.tiled_to_rowmajor(flat.cpu(), rows, K)
        assert torch.equal(back, t.cpu())
        pad = binding.tiled_to_rowmajor(flat.cpu(), (rows + 31) // 32 * 32, K)[rows:]
        assert torch.all(pad == 0)


@pytest.mark.parametrize("M,N,K,S", [
    (32, 256, 512, 1), (32, 256, 512, 2), (16, 3072, 2048, 0), (1, 128, 256, 1), (33, 128, 1024, 2),
    (64, 384, 768, 1), (5, 6144, 4096, 0), (32, 4096, 14336, 0),
    (32, 128256, 4096, 0),         # the LM head of the 8B shape (two weight tiles per workgroup)
    (40, 65664, 256, 1),           # the same form with two row tiles of activations
    # 33..64 rows, enough weight tiles: four tiles per workgroup sharing the activations through LDS
    (64, 5120, 1024, 0), (33, 25600, 256, 1), (64, 3200, 2304, 0), (50, 20480, 512, 2), (64, 5120, 5120, 0),
    (65, 128, 256, 1), (200, 256, 512, 1), (130, 384, 1024, 1), (4096, 128, 256, 1),
    # 256-row-tile GEMM: ragged last row tile, a last band of fewer than 8 row tiles, padding ids
    (3000, 4096, 256, 1), (2300, 5632, 512, 1),
])
def test_linear_tiled(M, N, K, S):
    a = rnd(60, (M, K)); w = rnd(61, (N, K), 0.05)
    ad, av = to_dev(a, "bf16"); wd, wv = to_dev(w, "bf16")
    if S == 0:
        S = binding.op_linear_splits("bf16", M, N, K, True)
    print("case: linear tiled", M, N, K, S, flush=True)
    out = binding.op_linear(binding.op_pack_tiled(ad), binding.op_pack_tiled(wd), S, tiled_shape=(M, N, K))
    out = out.cpu().numpy().astype(np.float64).sum(0)
    want = otf.linear(av, wv)
    np.testing.assert_allclose(out, want, rtol=0, atol=2e-5 * np.abs(want).max() + 1e-6)


@pytest.mark.parametrize("M,N,K", [(3000, 4096, 256), (2300, 5632, 512), (70, 128, 256), (130, 384, 1024), (300, 640, 512)])
def test_linear_accumulate_tiled(M, N, K):
    """x += a w^T in the GEMM's epilogue (ragged last row tile, padding workgroup ids)."""
    import torch
    a = rnd(160, (M, K)); w = rnd(161, (N, K), 0.05); x = rnd(162, (M, N), 3.0)
    ad, av = to_dev(a, "bf16"); wd, wv = to_dev(w, "bf16")
    print("case: linear accumulate", M, N, K, flush=True)
    xd = torch.from_numpy(x.astype(np.float32)).cuda()
    binding.op_linear_accumulate(binding.op_pack_tiled(ad), binding.op_pack_tiled(wd), xd, (M, N, K))
    want = x.astype(np.float32).astype(np.float64) + otf.linear(av, wv)
    np.testing.assert_allclose(xd.cpu().numpy(), want, rtol=0, atol=2e-5 * np.abs(want).max() + 1e-6)


@pytest.mark.parametrize("rows,Hq,Hkv,hd,K", [
    (19, 4, 2, 64, 256),           # few rows: the weight-streaming kernel
    (64, 8, 2, 128, 512),
    (2100, 32, 8, 128, 256),       # many rows: the 256-row-tile GEMM (ragged last tile)
    (6200, 12, 2, 128, 256),       # N = 2048
    (100, 4, 2, 64, 256),          # one ragged row tile, N = 512
    (300, 5, 1, 128, 512),         # N = 896: an odd number of 128-column workgroups
    (19, 32, 8, 128, 256),         # few rows, N = 6144: the row-range form, 24 weight rows per workgroup
    (32, 12, 2, 128, 512),         # N = 2048: 8 rows per workgroup
    (5, 64, 8, 128, 256),          # N = 10240: 40 rows per workgroup (ranges that end on a tile edge and inside one)
])
def test_linear_qkv_rope_fused(rows, Hq, Hkv, hd, K):
    """QKV projection + rotation + query / key / value stores in one kernel, against the oracle's
    linear layer and rotation."""
    import torch
    pg, base, n_pos = 64, 500000.0, 5000
    nq = (Hq + 2 * Hkv) * hd
    a = rnd(170, (rows, K)); w = rnd(171, (nq, K), 0.05)
    ad, av = to_dev(a, "bf16"); wd, wv = to_dev(w, "bf16")
    rng = np.random.default_rng(172)
    pos = rng.integers(0, n_pos, rows).astype(np.int32)
    pos[:3] = [0, 1, n_pos - 1]
    n_pages = -(-rows // pg) + 1
    slots = rng.permutation(n_pages * pg)[:rows]
    page, off = (slots // pg).astype(np.int32), (slots % pg).astype(np.int32)
    kp = torch.zeros((n_pages, Hkv, pg * hd), dtype=torch.bfloat16, device="cuda")
    vp = torch.zeros((n_pages, Hkv, pg * hd), dtype=torch.bfloat16, device="cuda")
    print("case: fused qkv rope", rows, Hq, Hkv, hd, K, flush=True)
    q = binding.op_linear_qkv_rope(
        binding.op_pack_tiled(ad), binding.op_pack_tiled(binding.interleave_qk_rows(wd, Hq, Hkv, hd)), rows, K,
        torch.from_numpy(pos).cuda(), torch.from_numpy(page).cuda(), torch.from_numpy(off).cuda(),
        Hq, Hkv, hd, pg, base, n_pos, kp, vp)
    full = otf.linear(av, wv).reshape(rows, Hq + 2 * Hkv, hd)
    wq = otf.rope(full[:, :Hq], pos, base)
    wk = otf.rope(full[:, Hq:Hq + Hkv], pos, base)
    wvv = full[:, Hq + Hkv:]
    tol = TOL["bf16"] * np.abs(full).max()
    np.testing.assert_allclose(q.float().cpu().numpy(), wq, rtol=0, atol=tol)
    ku, vu = binding.kv_pages_unpack(kp, vp, pg, hd)
    kh, vh = ku.float().cpu().numpy(), vu.float().cpu().numpy()
    np.testing.assert_allclose(kh[page, :, off, :], wk, rtol=0, atol=tol)
    np.testing.assert_allclose(vh[page, :, off, :], wvv, rtol=0, atol=tol)
    written = np.zeros((n_pages, pg), bool); written[page, off] = True
    assert np.all(kh.transpose(0, 2, 1, 3)[~written] == 0) and np.all(vh.transpose(0, 2, 1, 3)[~written] == 0)


@pytest.mark.parametrize("rows,Hq,Hkv,hd,pg,start", [(200, 4, 2, 64, 64, 0), (333, 4, 2, 128, 64, 37), (300, 8, 2, 64, 32, 17), (97, 6, 1, 128, 96, 90),
                                                     (1030, 8, 4, 128, 64, 1), (70, 4, 4, 32, 64, 50), (2100, 12, 2, 128, 64, 13)])
def test_linear_qkv_rope_consecutive_slots(rows, Hq, Hkv, hd, pg, start):
    """Keys and values of consecutive positions, as the session's passes write them (pages of any id, a first slot inside a
    16-slot group, page ends inside a tile): every slot has the bits of the same product with its slots shuffled
    (which goes by single values), and the others stay zero."""
    import torch
    K, base = 256, 1.0e4
    nq = (Hq + 2 * Hkv) * hd
    a = binding.op_pack_tiled(to_dev(rnd(940, (rows, K)), "bf16")[0])
    w = binding.op_pack_tiled(to_dev(rnd(941, (nq, K), 0.05), "bf16")[0])
    n_pages = -(-(start + rows) // pg)
    rng = np.random.default_rng(942)
    ids = rng.permutation(n_pages)
    at = start + np.arange(rows)
    lines = ids[at // pg] * pg + at % pg
    mixed = rng.permutation(n_pages * pg)[:rows]

    def run(slots):
        t = lambda x: torch.from_numpy(x.astype(np.int32)).cuda()  # noqa: E731
        kp = torch.zeros((n_pages, Hkv, pg * hd), dtype=torch.bfloat16, device="cuda")
        vp = torch.zeros_like(kp)
        q = binding.op_linear_qkv_rope(a, w, rows, K, t(at), t(slots // pg), t(slots % pg), Hq, Hkv, hd, pg, base, start + rows, kp, vp)
        k, v = (x.transpose(1, 2).reshape(-1, Hkv, hd) for x in binding.kv_pages_unpack(kp, vp, pg, hd))
        rest = np.setdiff1d(np.arange(n_pages * pg), slots)
        assert not k[rest].any() and not v[rest].any()
        return q, k[slots], v[slots]

    print("case: qkv rope, consecutive slots", rows, Hq, Hkv, hd, pg, start, flush=True)
    for name, x, y in zip(("queries", "keys", "values"), run(lines), run(mixed)):
        assert x.any() and torch.equal(x, y), name


@pytest.mark.parametrize("M,N,K", [(32, 256, 512), (7, 14336, 4096), (64, 128, 256), (150, 256, 512),
                                   (3000, 2048, 512), (2070, 2944, 256), (65, 384, 256),
                                   (50, 27648, 512), (64, 20480, 256),
                                   # the row-range form: 56, 24, 8 and 48 weight rows per workgroup
                                   (32, 14336, 256), (17, 6144, 512), (1, 2048, 256), (30, 12288, 256)])
def test_linear_swiglu_tiled(M, N, K):
    a = rnd(62, (M, K)); wg = rnd(63, (N, K), 0.05); wu = rnd(64, (N, K), 0.05)
    ad, av = to_dev(a, "bf16"); gd, gv = to_dev(wg, "bf16"); ud, uv = to_dev(wu, "bf16")
    print("case: swiglu tiled", M, N, K, flush=True)
    flat = binding.op_linear_swiglu(binding.op_pack_tiled(ad), binding.op_pack_tiled(gd),
                                    binding.op_pack_tiled(ud), tiled_shape=(M, N, K))
    out = binding.tiled_to_rowmajor(flat.cpu(), M, N).float().numpy()
    want = otf.silu(otf.linear(av, gv)) * otf.linear(av, uv)
    np.testing.assert_allclose(out, want, rtol=0, atol=TOL["bf16"] * np.abs(want).max())


# A few hundred rows: the 128-row GEMM tiles with one, two and four weight tiles per workgroup (one and
# more groups of four units of K, a last workgroup with few rows, the last row count that takes each
# form and the first past it).
@pytest.mark.parametrize("M,N,K", [(65, 4096, 256), (128, 4096, 768), (129, 4096, 256), (256, 4096, 1280), (257, 4096, 768),
                                   (300, 4096, 512), (512, 4096, 256), (513, 4096, 512), (1023, 2048, 768)])
def test_linear_few_hundred_rows(M, N, K):
    test_linear_tiled(M, N, K, 1)
    test_linear_accumulate_tiled(M, N, K)


@pytest.mark.parametrize("M,N,K", [(65, 2048, 256), (128, 2048, 768), (130, 4096, 256), (200, 2048, 1280), (300, 8192, 256)])
def test_linear_swiglu_few_hundred_rows(M, N, K):
    test_linear_swiglu_tiled(M, N, K)


@pytest.mark.parametrize("rows,Hq,Hkv,hd,K", [(65, 8, 2, 64, 256), (100, 32, 8, 64, 512), (200, 32, 8, 128, 256), (330, 32, 8, 128, 768),
                                              (700, 12, 2, 128, 256)])
def test_linear_qkv_rope_few_hundred_rows(rows, Hq, Hkv, hd, K):
    test_linear_qkv_rope_fused(rows, Hq, Hkv, hd, K)


@pytest.mark.parametrize("N,K,Hq,Hkv,rows,forms", [
    (4096, 768, 16, 8, (100, 200, 300, 600, 3000), ((64, 32), (128, 32), (128, 64), (128, 128), (256, 128))),
    (5120, 768, 20, 10, (192, 3000), ((64, 64), (256, 128))),
    (4096, 12288, 16, 8, (300, 3000), ((96, 64), (256, 128)))])
def test_many_row_gemm_forms_give_the_same_bits(N, K, Hq, Hkv, rows, forms):
    """Rows alone, with more rows and in a chunk, which are workgroups of every shape (rows x columns) that the plain and
    the rotary products take: the same bits in every output form, and every form twice."""
    import torch
    assert tuple(binding.op_gemm_plan(M, N, K)[:2] for M in rows) == forms
    w = binding.op_pack_tiled(to_dev(rnd(550, (N, K), 0.05), "bf16")[0])
    w2 = binding.op_pack_tiled(to_dev(rnd(551, (N, K), 0.05), "bf16")[0])
    hd, pg = 128, 64                                    # (Hq + 2 Hkv) hd = N
    a = to_dev(rnd(552, (rows[-1], K)), "bf16")[0]
    x0 = to_dev(rnd(553, (rows[-1], N)), "f32")[0]

    def outputs(M):
        am = binding.op_pack_tiled(a[:M].contiguous())
        at = torch.arange(M, dtype=torch.int32, device="cuda")
        kp = torch.zeros((-(-M // pg), Hkv, pg * hd), dtype=torch.bfloat16, device="cuda")
        vp = torch.zeros_like(kp)
        q = binding.op_linear_qkv_rope(am, w, M, K, at, at // pg, at % pg, Hq, Hkv, hd, pg, 1.0e4, M, kp, vp)
        act = binding.op_linear_swiglu(am, w, w2, tiled_shape=(M, N, K))
        out = [binding.op_linear(am, w, 1, tiled_shape=(M, N, K))[0], binding.op_linear_accumulate(am, w, x0[:M].clone(), (M, N, K)),
               binding.tiled_to_rowmajor(act, M, N), q] + list(binding.kv_pages_unpack(kp, vp, pg, hd))
        out[4:] = [t.transpose(1, 2).reshape(-1, Hkv, hd)[:M] for t in out[4:]]
        return out

    names = ("sums", "residual", "swiglu", "queries", "keys", "values")
    full = outputs(rows[-1])
    for M in rows:
        print("case: GEMM forms", N, K, M, flush=True)
        one, two = outputs(M), outputs(M)
        for name, x, y, z in zip(names, one, two, full):
            assert torch.equal(x, y), (name, M, "run to run")
            assert torch.equal(x, z[:M]), (name, M)


def test_gemm_weights_in_bursts():
    """The forms that ask for the weights of four units at once (128, 192 and 256 rows x 64 columns), full and ragged, and the ones beside
    them: the bits of the 256 x 128 workgroups in every output form, over a K that is several bursts and over one that is just long enough."""
    test_many_row_gemm_forms_give_the_same_bits(4096, 4096, 16, 8, (449, 512, 520, 768, 1000, 3000),
                                                ((128, 64), (128, 64), (192, 64), (192, 64), (256, 64), (256, 128)))
    test_many_row_gemm_forms_give_the_same_bits(2048, 2304, 8, 4, (1000, 1100, 5000), ((128, 64), (128, 128), (256, 128)))


@pytest.mark.parametrize("M,N,K", [(128, 8192, 256), (129, 4096, 512), (65, 5120, 256), (129, 5120, 768), (192, 5120, 256), (193, 5120, 256)])
def test_linear_64_row_workgroups(M, N, K):
    """GEMM workgroups of two waves (64 rows x 32 or 64 columns): full and ragged last workgroups, the last row
    count that takes the form and the first past it."""
    test_linear_tiled(M, N, K, 1)
    test_linear_accumulate_tiled(M, N, K)


@pytest.mark.parametrize("M,N", [(289, 4096), (384, 4096), (193, 5120)])
def test_gemm_96_row_workgroups(M, N):
    """GEMM workgroups of three waves (96 rows x 64 columns; one wave brings no weights), over a K that takes them: a ragged
    and a full last workgroup, in the three plain output forms."""
    K = 12288
    test_linear_tiled(M, N, K, 1)
    test_linear_accumulate_tiled(M, N, K)
    test_linear_qkv_rope_fused(M, N // 256, N // 512, 128, K)


@pytest.mark.parametrize("M,K", [(100, 256), (257, 256), (320, 768), (321, 512), (384, 256), (385, 256)])
def test_linear_swiglu_wide_workgroups(M, K):
    """The SwiGLU form with a wave per row tile (10 and 12 waves; waves past the last row tile), its neighbours, and
    the single row tile whose weights bypass L2: against the oracle, and a row has the bits that it has in any
    other launch."""
    import torch
    N = 14336
    test_linear_swiglu_tiled(M, N, K)
    a = to_dev(rnd(62, (M, K)), "bf16")[0]
    wg, wu = (binding.op_pack_tiled(to_dev(rnd(s, (N, K), 0.05), "bf16")[0]) for s in (63, 64))
    run = lambda m: binding.tiled_to_rowmajor(binding.op_linear_swiglu(binding.op_pack_tiled(a[:m].contiguous()), wg, wu, tiled_shape=(m, N, K)), m, N)  # noqa: E731
    full = run(M)
    assert torch.equal(full, run(M)) and torch.equal(full[:70], run(70)) and torch.equal(full[:130], run(min(M, 130))[:130])


def test_scoring_size_gemms_on_sampled_rows():
    """The many-row GEMMs at the sizes one scoring chunk of the 8B shape launches (8192 rows):
    gate/up + SwiGLU 8192 x 14336 x 4096, down with the residual update 8192 x 4096 x 14336, QKV
    with rotation and page stores 8192 x 6144 x 4096.  The oracle computes 24 sampled rows of each
    (first, last, tile borders, random ones); every column of those rows is compared."""
    import torch
    M = 8192
    rng = np.random.default_rng(180)
    rows_s = np.unique(np.concatenate([[0, 31, 32, 255, 256, M - 257, M - 1], rng.integers(0, M, 17)]))
    # gate/up + SwiGLU
    d, F = 4096, 14336
    a = rnd(181, (M, d)); wg = rnd(182, (F, d), 0.02); wu = rnd(183, (F, d), 0.02)
    ad, av = to_dev(a, "bf16"); gd, gv = to_dev(wg, "bf16"); ud, uv = to_dev(wu, "bf16")
    print("case: scoring-size swiglu", flush=True)
    flat = binding.op_linear_swiglu(binding.op_pack_tiled(ad), binding.op_pack_tiled(gd), binding.op_pack_tiled(ud),
                                    tiled_shape=(M, F, d))
    act = binding.tiled_to_rowmajor(flat.cpu(), M, F)
    want = otf.silu(otf.linear(av[rows_s], gv)) * otf.linear(av[rows_s], uv)
    np.testing.assert_allclose(act[rows_s].float().numpy(), want, rtol=0, atol=TOL["bf16"] * np.abs(want).max())
    del gd, ud, flat
    # down projection adding to the residual stream; its input is the product above
    wd_ = rnd(184, (d, F), 0.02); x = rnd(185, (M, d), 2.0)
    dd, dv = to_dev(wd_, "bf16")
    print("case: scoring-size accumulate", flush=True)
    xd = torch.from_numpy(x.astype(np.float32)).cuda()
    actd = act.cuda()
    binding.op_linear_accumulate(binding.op_pack_tiled(actd), binding.op_pack_tiled(dd), xd, (M, d, F))
    want = x[rows_s].astype(np.float32).astype(np.float64) + otf.linear(act[rows_s].float().numpy(), dv)
    np.testing.assert_allclose(xd.cpu().numpy()[rows_s], want, rtol=0, atol=2e-5 * np.abs(want).max() + 1e-6)
    del dd, actd, xd
    # QKV + rotation + page stores
    Hq, Hkv, hd, pg, base, n_pos = 32, 8, 128, 64, 500000.0, 5120
    nq = (Hq + 2 * Hkv) * hd
    w = rnd(186, (nq, d), 0.02)
    wd2, wv = to_dev(w, "bf16")
    pos = rng.integers(0, n_pos, M).astype(np.int32)
    slots = rng.permutation((M // pg + 2) * pg)[:M]
    page, off = (slots // pg).astype(np.int32), (slots % pg).astype(np.int32)
    kp = torch.zeros((M // pg + 2, Hkv, pg * hd), dtype=torch.bfloat16, device="cuda")
    vp = torch.zeros_like(kp)
    print("case: scoring-size fused qkv rope", flush=True)
    q = binding.op_linear_qkv_rope(
        binding.op_pack_tiled(ad), binding.op_pack_tiled(binding.interleave_qk_rows(wd2, Hq, Hkv, hd)), M, d,
        torch.from_numpy(pos).cuda(), torch.from_numpy(page).cuda(), torch.from_numpy(off).cuda(),
        Hq, Hkv, hd, pg, base, n_pos, kp, vp)
    full = otf.linear(av[rows_s], wv).reshape(len(rows_s), Hq + 2 * Hkv, hd)
    tol = TOL["bf16"] * np.abs(full).max()
    np.testing.assert_allclose(q[torch.from_numpy(rows_s).cuda()].float().cpu().numpy(),
                               otf.rope(full[:, :Hq], pos[rows_s], base), rtol=0, atol=tol)
    ku, vu = binding.kv_pages_unpack(kp, vp, pg, hd)
    kh, vh = ku.float().cpu().numpy(), vu.float().cpu().numpy()
    np.testing.assert_allclose(kh[page[rows_s], :, off[rows_s], :], otf.rope(full[:, Hq:Hq + Hkv], pos[rows_s], base), rtol=0, atol=tol)
    np.testing.assert_allclose(vh[page[rows_s], :, off[rows_s], :], full[:, Hq + Hkv:], rtol=0, atol=tol)


def test_tiled_outputs_of_rmsnorm_and_attention():
    import torch
    for rows, d in [(37, 256), (1001, 512)]:      # the second: many rows, dealt to the XCDs in contiguous ranges
        x = rnd(65, (rows, d)); g = 1 + rnd(66, (d,), 0.1); p = rnd(67, (1, rows, d))
        gd, gv = to_dev(g, "bf16")
        h_plain = binding.op_add_rmsnorm(torch.from_numpy(x.copy()).cuda(), torch.from_numpy(p).cuda(), gd, 1e-6)
        xt = torch.from_numpy(x.copy()).cuda()
        h_tiled = binding.op_add_rmsnorm(xt, torch.from_numpy(p).cuda(), gd, 1e-6, tiled=True)
        assert torch.equal(binding.tiled_to_rowmajor(h_tiled.cpu(), rows, d), h_plain.cpu())
        want_x = x.astype(np.float64) + p[0]
        np.testing.assert_allclose(xt.cpu().numpy(), want_x, rtol=0, atol=1e-6)
        want_h = otf.rmsnorm(want_x, gv, 1e-6)
        np.testing.assert_allclose(h_plain.float().cpu().numpy(), want_h, rtol=0, atol=TOL["bf16"] * 4)
    # attention output, [B][Hq*hd] tiled
    B, Hq, Hkv, hd, pg, P, t = 5, 4, 2, 64, 16, 40, 9
    kpd, vpd, _, _ = make_pools("bf16", 3, Hkv, pg, hd, 70)
    ksd, vsd, _, _ = make_pools("bf16", B, Hkv, pg, hd, 72)
    table = torch.arange(B, dtype=torch.int32, device="cuda").reshape(B, 1)
    qd, _ = to_dev(rnd(74, (B, Hq, hd)), "bf16")
    o_plain = binding.op_attention_decode(qd, kpd, vpd, ksd, vsd, table, P, t, pg)
    o_tiled = binding.op_attention_decode(qd, kpd, vpd, ksd, vsd, table, P, t, pg, out_tiled=True)
    assert torch.equal(binding.tiled_to_rowmajor(o_tiled.cpu(), B, Hq * hd), o_plain.cpu().reshape(B, Hq * hd))


# ---------------------------------------------------------------- MFMA prefill / scoring attention
def prefill_case(Hq, Hkv, hd, P, seqs, stride=1, seed=90, out_tiled=False, item_rows=64, qscale=1.0, plant=()):
    """seqs: list of (pos_start, n_rows); pos_start < P means a prefix chunk (keys = prefix
    only, P grows to cover it), pos_start >= P a scored suffix starting at P.  plant: (row, head,
    key position) tuples: that key (a position the row can see) becomes 3 q[row, head].
    Returns (worst relative L2 error over the compared rows, errors of the planted rows)."""
    import torch
    pg = 64
    scoring = any(p0 >= P for p0, _ in seqs)
    n_pre = -(-P // pg)
    kpd, vpd, kpv, vpv = make_pools("bf16", n_pre, Hkv, pg, hd, seed)
    per = max(-(-max(n for _, n in seqs) // pg), 1)
    ksd, vsd, ksv, vsv = make_pools("bf16", len(seqs) * per, Hkv, pg, hd, seed + 2)
    table = np.random.default_rng(seed).permutation(len(seqs) * per).astype(np.int32).reshape(len(seqs), per)
    rows = sum(n for _, n in seqs)
    q = rnd(seed + 4, (rows, Hq, hd), qscale); qd, qv = to_dev(q, "bf16")
    G = Hq // Hkv
    seq_of_row = np.concatenate([np.full(n, si) for si, (_, n) in enumerate(seqs)]) if rows else np.zeros(0, int)
    for r, a, kpos in plant:
        if kpos < P:
            plant_key(kpv, vpv, kpd, vpd, kpos // pg, a // G, kpos % pg, qv[r, a], 3.0 / qscale, "bf16")
        else:
            j = kpos - P
            plant_key(ksv, vsv, ksd, vsd, table[seq_of_row[r], j // pg], a // G, j % pg, qv[r, a], 3.0 / qscale, "bf16")
    items, r0 = [], 0
    for si, (p0, n) in enumerate(seqs):
        for j in range(0, n, item_rows):
            items.append([r0 + j, min(item_rows, n - j), p0 + j, si if scoring else -1])
        r0 += n
    it = torch.tensor(items, dtype=torch.int32, device="cuda")
    print("case: prefill attention", Hq, Hkv, hd, P, seqs, plant, flush=True)
    out = binding.op_attention_prefill(qd, it, kpd, vpd, ksd if scoring else None, vsd if scoring else None,
                                       torch.from_numpy(table).cuda() if scoring else None, P, pg, out_tiled)
    if out_tiled:
        out = binding.tiled_to_rowmajor(out.cpu(), rows, Hq * hd).reshape(rows, Hq, hd)
    out = out.float().cpu().numpy()
    pos_of_row = np.concatenate([p0 + np.arange(n) for p0, n in seqs]) if rows else np.zeros(0, int)

    def want_row(r, a):
        si, pos, c = seq_of_row[r], pos_of_row[r], a // G
        keys = [kpv[:, c].reshape(-1, hd)[:min(P, pos + 1)]]
        vals = [vpv[:, c].reshape(-1, hd)[:min(P, pos + 1)]]
        if pos >= P:
            keys.append(ksv[table[si], c].reshape(-1, hd)[:pos - P + 1])
            vals.append(vsv[table[si], c].reshape(-1, hd)[:pos - P + 1])
        return otf.attention_one(qv[r, a], np.concatenate(keys), np.concatenate(vals))

    worst = 0.0
    for r in range(rows):
        for a in range(Hq):
            if (r * Hq + a) % stride == 0:
                worst = max(worst, rel_l2(out[r, a], want_row(r, a)))
    return worst, [rel_l2(out[r, a], want_row(r, a)) for r, a, _ in plant]


@pytest.mark.parametrize("Hq,Hkv,hd,P,seqs,stride,plant", [
    (8, 2, 128, 200, [(0, 200)], 1, [(199, 7, 150), (70, 0, 70)]),          # first prefill chunk, causal from position 0
    (8, 2, 64, 330, [(130, 200)], 1, [(199, 3, 5), (100, 6, 229)]),         # later chunk: earlier keys + own diagonal
    (32, 8, 128, 4096, [(2048, 2048)], 211, [(2047, 31, 4094), (1000, 5, 2000), (3, 12, 100)]),   # 8B shape, second half of the prefix
    (8, 2, 128, 150, [(150, 70), (150, 33), (150, 1)], 1, [(69, 1, 218), (90, 4, 149), (103, 7, 150)]),  # scoring: ragged suffixes
    (40, 8, 128, 1000, [(1000, 100), (1000, 64)], 7, [(99, 39, 999), (163, 20, 1063)]),            # 5 query heads per KV head
    (32, 8, 128, 4096, [(4096, 1024)] * 3, 1531, [(1023, 0, 5119), (2047, 31, 4000), (3071, 9, 5000), (2500, 17, 4500)]),  # reranking shape
    (4, 4, 64, 1, [(1, 65)], 1, [(64, 2, 65)]),
])
def test_attention_prefill_mfma(Hq, Hkv, hd, P, seqs, stride, plant):
    """Every compared row within the relative bound, and rows one of whose keys (late in the
    prefix, in the row's own suffix page, on its own diagonal) decides the output."""
    worst, planted = prefill_case(Hq, Hkv, hd, P, seqs, stride, plant=plant)
    assert worst < ATT_REL["bf16"], worst
    assert max(planted) < ATT_REL["bf16"], planted


@pytest.mark.parametrize("item_rows", [32, 48, 17])
def test_attention_prefill_item_sizes(item_rows):
    """Items shorter than 64 positions: the second half of the workgroup has fewer rows or none."""
    worst, _ = prefill_case(8, 2, 128, 150, [(150, 130), (150, 33)], item_rows=item_rows)
    assert worst < ATT_REL["bf16"], worst
    worst, _ = prefill_case(8, 2, 64, 200, [(0, 200)], item_rows=item_rows)
    assert worst < ATT_REL["bf16"], worst


def prefill_kernel(Hq, Hkv, hd, P, seqs):
    """The kernel that prefill_case runs for these sizes."""
    stride = -(-max(n for _, n in seqs) // 64) if any(p0 >= P for p0, _ in seqs) else 0
    return binding.op_attention_prefill_plan(sum(-(-n // 64) for _, n in seqs), Hq, Hkv, hd, 64, P, stride)[0]


@pytest.mark.parametrize("Hq,Hkv,hd,P,seqs,stride,kernel", [
    # scoring and adding waves: two pages a step, an odd number of pages, a prefix that ends inside its last
    # page's first block, three query heads for two per workgroup; more of a prefix, scored suffixes
    (8, 2, 128, 2593, [(2593, 40), (2593, 1)], 3, "pair"), (6, 2, 128, 2700, [(2700, 50)], 3, "pair"), (8, 2, 64, 2626, [(2596, 30)], 1, "pair"),
    # a second round of them: several sequences behind a long prefix, a late part of a prefix
    (32, 8, 128, 3100, [(3100, 64)] * 10, 97, "pair"), (32, 8, 64, 3130, [(2600, 530)], 211, "pair"),
    # item counts at the ends of the rounds, and the first past them
    (32, 8, 128, 3112, [(2600, 512)], 401, "pair"), (32, 8, 64, 3113, [(2600, 513)], 401, "pair"), (32, 8, 128, 3624, [(2600, 1024)], 1601, "pair"),
    (32, 8, 64, 3625, [(2600, 1025)], 1601, "whole"),
    # two waves per head: suffixes of one page each behind prefixes that end in a page's first block, its second, at its end
    (32, 8, 128, 2570, [(2570, 64)] * 10, 97, "split"), (32, 8, 64, 1965, [(1965, 64)] * 10, 97, "split"), (32, 8, 64, 1920, [(1920, 33)] * 16, 61, "split"),
    # ... three, five and eight query heads for four per workgroup, items of one half
    (6, 2, 128, 700, [(700, 20)] * 40, 61, "split"), (10, 2, 64, 741, [(741, 64)] * 25, 211, "split"), (16, 2, 128, 129, [(129, 40)] * 20, 97, "split"),
    (64, 8, 128, 500, [(200, 300)], 301, "split"),
    # ... page ids in registers of 64: a prefix and suffixes that go through two of them
    (8, 1, 128, 3000, [(3000, 1200), (3000, 1000)], 401, "split"), (8, 1, 64, 2000, [(2000, 2200)], 401, "split"),
    # whole pages only and suffixes that end early; rows at the prefix's begin: waves whose blocks no row sees
    (8, 2, 128, 2560, [(2560, 33)], 1, "pair"), (8, 2, 64, 2561, [(0, 70)], 1, "pair"),
    # page ids in registers of 64: a suffix that goes through two of them, a prefix that goes through three
    (2, 1, 128, 100, [(100, 4300)], 97, "pair"), (2, 1, 64, 4032, [(4032, 130)], 7, "pair"), (4, 2, 128, 8250, [(8250, 20)], 1, "pair"),
])
def test_attention_prefill_key_groups(Hq, Hkv, hd, P, seqs, stride, kernel):
    assert prefill_kernel(Hq, Hkv, hd, P, seqs) == kernel
    worst, _ = prefill_case(Hq, Hkv, hd, P, seqs, stride)
    assert worst < ATT_REL["bf16"], worst


@pytest.mark.parametrize("hd,P,rows,kernels", [
    (128, 300, 100, ("pair", "pair", "split", "whole", "whole")), (64, 300, 100, ("pair", "pair", "split", "whole", "whole")),
    (128, 2700, 70, ("pair", "pair", "split", "whole", "whole")), (64, 2700, 70, ("pair", "pair", "pair", "whole", "whole")),
    (128, 4097, 33, ("pair", "pair", "pair", "pair", "whole")), (128, 2050, 40, ("pair", "pair", "pair", "split", "whole")),
    (128, 8200, 40, ("pair", "pair", "pair", "pair", "whole"))])
def test_attention_prefill_rows_do_not_depend_on_the_launch(hd, P, rows, kernels):
    """A candidate's rows scored alone, with a few others and in a full chunk, which take scoring and adding waves, two waves
    per head and whole items: the same bits.  Some keys outgrow the softmax's reference far into the walk, in every
    place of a step of four blocks."""
    import torch
    Hq, Hkv, pg, n = 32, 8, 64, 24
    g = torch.Generator(device="cuda")
    g.manual_seed(7 * P + hd)
    normal = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)  # noqa: E731
    per, n_pre = -(-rows // pg), -(-P // pg)
    k, v = normal(n_pre, Hkv, pg, hd), normal(n_pre, Hkv, pg, hd)
    for page, key in [(1, 5), (2, 40), (3, 63), (n_pre - 2, 33)]:
        k[page, :, key] *= 8
    kp, vp = binding.kv_pages_pack(k, v)
    ks, vs = binding.kv_pages_pack(normal(n * per, Hkv, pg, hd), normal(n * per, Hkv, pg, hd))
    table = torch.randperm(n * per, generator=g, device="cuda").to(torch.int32).reshape(n, per)
    q = normal(n * rows, Hq, hd) * 2

    def score(cands):
        items = [[i * rows + j, min(64, rows - j), P + j, c] for i, c in enumerate(cands) for j in range(0, rows, 64)]
        rq = torch.cat([q[c * rows: (c + 1) * rows] for c in cands])
        out = binding.op_attention_prefill(rq, torch.tensor(items, dtype=torch.int32, device="cuda"), kp, vp, ks, vs, table, P, pg)
        return out.view(torch.int16).reshape(len(cands), rows, Hq, hd)

    print("case: prefill rows alone and together", hd, P, rows, flush=True)
    assert tuple(prefill_kernel(Hq, Hkv, hd, P, [(P, rows)] * m) for m in (1, 4, 8, 14, n)) == kernels
    full = score(list(range(n)))
    assert torch.equal(score(list(range(n))), full)
    assert not torch.isnan(full.view(torch.bfloat16)).any()
    for cands in ([3], [5, 3, 17, 0], list(range(n - 1, n - 9, -1)), list(range(14))):
        assert torch.equal(score(cands), score(cands))
        assert torch.equal(score(cands), full[cands]), (len(cands), "candidates")


def test_attention_prefill_tiled_output_matches():
    a, _ = prefill_case(8, 2, 128, 100, [(100, 40), (100, 9)], out_tiled=True)
    assert a < ATT_REL["bf16"], a


@pytest.mark.parametrize("qscale", [8.0, 0.01])
def test_attention_with_peaked_and_flat_softmax(qscale):
    """Scores with a standard deviation of ~90 (one key takes nearly all the weight, the running
    maximum jumps far past the lazy rescale threshold several times) and of ~0.1 (uniform
    weights), on both MFMA attention kernels."""
    worst, _, _ = attention_case("bf16", 9, 8, 2, 128, 64, 700, 130, qscale=qscale, stride=3)
    assert worst < 2 * ATT_REL["bf16"], worst
    worst, _, _ = attention_case("bf16", 4, 4, 4, 64, 64, 0, 257, qscale=qscale)
    assert worst < 2 * ATT_REL["bf16"], worst
    # short contexts: a workgroup per candidate and KV head (0), split keys; many rows: four row blocks per prefix item
    for B, P, t, splits in ((9, 500, 130, 0), (9, 500, 130, 3), (4, 0, 257, 1), (64, 500, 130, 3)):
        worst, _, _ = attention_case("bf16", B, 8, 2, 128, 64, P, t, splits=splits, qscale=qscale, stride=1 + B // 4)
        assert worst < 2 * ATT_REL["bf16"], (worst, B, splits)
    worst, _ = prefill_case(8, 2, 128, 150, [(150, 130)], qscale=qscale, stride=3)
    assert worst < 2 * ATT_REL["bf16"], worst
    for Hq, Hkv, hd, seqs, kernel in ((32, 8, 128, [(150, 64)] * 10, "split"), (32, 8, 64, [(150, 64)] * 40, "whole"), (40, 8, 128, [(150, 40)] * 20, "rest")):
        assert prefill_kernel(Hq, Hkv, hd, 150, seqs) == kernel
        worst, _ = prefill_case(Hq, Hkv, hd, 150, seqs, qscale=qscale, stride=211)
        assert worst < 2 * ATT_REL["bf16"], (worst, kernel)


def test_mfma_probe_counts_what_it_claims():
    """All-ones operands: every accumulator element gains 16 per MFMA, so a thread's 8 tiles x 16
    registers sum to 8 * 16 * 16 * iters."""
    import torch
    n_wg, iters = 3, 5
    ops = torch.ones(n_wg * 256 * 48, dtype=torch.bfloat16, device="cuda")
    out = torch.empty(n_wg * 256, dtype=torch.float32, device="cuda")
    lib = binding.load_library()
    assert lib.mc_op_mfma_probe(None, ops.data_ptr(), out.data_ptr(), n_wg, iters) == 0
    torch.cuda.synchronize()
    assert torch.all(out == 8 * 16 * 16 * iters)
    assert binding.op_mfma_probe(ops, n_wg, iters) == n_wg * 4 * iters * 8 * 32768.0


def _poison(n):
    """Leave NaN where the next buffer of n bf16 values is allocated from."""
    import torch
    t = torch.full((n,), float("nan"), dtype=torch.bfloat16, device="cuda")
    del t


def _padding_of(flat, rows, K):
    return binding.tiled_to_rowmajor(flat, (rows + 31) // 32 * 32, K)[rows:]


@pytest.mark.parametrize("rows,d", [(1, 64), (31, 256), (33, 4096), (300, 2048), (2050, 1024), (5, 16448)])
def test_norm_writes_its_padding_rows(rows, d):
    import torch
    x = to_dev(rnd(920, (rows, d)), "f32")[0]
    _poison((rows + 31) // 32 * 32 * d)
    h = binding.op_add_rmsnorm(x, None, torch.ones(d, dtype=torch.bfloat16, device="cuda"), 1e-6, tiled=True)
    assert not h.isnan().any() and not _padding_of(h, rows, d).any()
    want = x.double() / torch.sqrt((x.double() ** 2).mean(-1, keepdim=True) + 1e-6)
    assert rel_l2(binding.tiled_to_rowmajor(h, rows, d).double().cpu().numpy(), want.cpu().numpy()) < TOL["bf16"]


# the tile per workgroup, the row ranges, shared activations, two row tiles, and the GEMM's forms
@pytest.mark.parametrize("M,N,K", [(5, 256, 512), (17, 6144, 256), (50, 20480, 256), (40, 256, 256), (70, 14336, 256), (100, 2048, 256),
                                   (150, 8192, 256), (270, 14336, 256), (330, 14336, 256), (601, 14336, 256)])
def test_swiglu_writes_its_padding_rows(M, N, K):
    a, wg, wu = (binding.op_pack_tiled(to_dev(rnd(s, (n, K), 0.1), "bf16")[0]) for s, n in ((921, M), (922, N), (923, N)))
    _poison((M + 31) // 32 * 32 * N)
    out = binding.op_linear_swiglu(a, wg, wu, tiled_shape=(M, N, K))
    assert not out.isnan().any() and not _padding_of(out, M, N).any()


@pytest.mark.parametrize("B,Hq,Hkv,hd,pg,P,t,splits", [
    (8, 32, 8, 64, 64, 777, 37, 0), (1, 8, 2, 128, 64, 300, 5, 0), (33, 8, 2, 128, 64, 300, 5, 0),     # a workgroup per candidate and KV head
    (5, 8, 2, 128, 64, 20, 0, 0), (9, 8, 4, 64, 64, 0, 30, 0),                                         # ... prefix, suffix alone
    (8, 32, 8, 64, 64, 777, 37, 2), (1, 8, 2, 128, 64, 300, 5, 1), (33, 8, 2, 128, 64, 300, 5, 3),     # merged partial states
    (64, 32, 8, 128, 64, 700, 33, 4),                                                                  # ... four row blocks per prefix item
    (3, 8, 2, 64, 64, 3000, 1, 64),                                                                    # more of them than one batch
    (5, 8, 2, 128, 64, 20, 0, 1), (9, 8, 4, 64, 64, 0, 30, 1), (57, 32, 8, 128, 64, 100, 0, 1),        # one: the items write
    (5, 8, 2, 96, 64, 100, 9, 0), (7, 4, 2, 64, 16, 33, 4, 0)])                                        # the generic kernel
def test_decode_attention_writes_its_padding_rows(B, Hq, Hkv, hd, pg, P, t, splits):
    import torch
    kp, vp, _, _ = make_pools("bf16", max(1, -(-P // pg)), Hkv, pg, hd, 924)
    per = max(1, -(-t // pg))
    ks, vs, _, _ = make_pools("bf16", B * per, Hkv, pg, hd, 925)
    table = torch.arange(B * per, dtype=torch.int32, device="cuda").reshape(B, per)
    q = to_dev(rnd(926, (B, Hq, hd)), "bf16")[0]
    run = lambda tiled: binding.op_attention_decode(q, kp if P else None, vp if P else None, ks, vs, table, P, t, pg, splits, out_tiled=tiled)  # noqa: E731
    _poison((B + 31) // 32 * 32 * Hq * hd)
    out = run(True)
    assert not out.isnan().any() and not _padding_of(out, B, Hq * hd).any()
    assert torch.equal(binding.tiled_to_rowmajor(out, B, Hq * hd).reshape(B, Hq, hd), run(False))


def _tile_calls(n):
    """Row ranges of one tile that several calls fill, 16 bytes a row further each: (first row, rows)."""
    return [(0, n), (n, 3), (n + 3, 32 - n - 3 - 2)]


def _assert_tile(out, want, K, written):
    """The rows written hold `want`, the others of the two tiles and everything past them their old values."""
    got = binding.tiled_to_rowmajor(out, 64, K)
    import torch
    assert torch.equal(got[:written], want[:written]) and torch.all(got[written:] == -7)


def test_tiled_outputs_leave_rows_that_are_not_theirs():
    """The entry points without _tiled in their name store their rows and nothing else: the padding rows of a caller's
    buffer stay, and one 32-row tile may be filled by several calls."""
    import torch
    lib = binding.load_library()
    d, n = 512, 11
    dev = lambda seed, shape, scale=1.0: to_dev(rnd(seed, shape, scale), "bf16")[0]  # noqa: E731
    print("case: tiled outputs of several calls", flush=True)
    for width in (d, 16448):                                            # norm: by quads, one row after another
        x, gain = to_dev(rnd(960, (30, width)), "f32")[0], dev(961, (width,))
        want = binding.op_add_rmsnorm(x, None, gain, 1e-6)
        out = torch.full((64 * width,), -7.0, dtype=torch.bfloat16, device="cuda")
        for r0, rows in _tile_calls(n):
            assert lib.mc_op_add_rmsnorm(None, 1, rows, width, x[r0:].data_ptr(), None, 0, gain.data_ptr(), 1e-6, out.data_ptr() + 16 * r0, 1) == 0
        _assert_tile(out, want, width, 30)
    a = dev(962, (30, 256))
    for N in (128, 14336):                                             # SwiGLU: a tile and a range of rows per workgroup
        wg, wu = (binding.op_pack_tiled(dev(s, (N, 256), 0.1)) for s in (963, 964))
        want = binding.tiled_to_rowmajor(binding.op_linear_swiglu(binding.op_pack_tiled(a), wg, wu, tiled_shape=(30, N, 256)), 30, N)
        out = torch.full((64 * N,), -7.0, dtype=torch.bfloat16, device="cuda")
        for r0, rows in _tile_calls(n):
            at = binding.op_pack_tiled(a[r0:r0 + rows].contiguous())
            assert lib.mc_op_linear_swiglu(None, 1, rows, N, 256, at.data_ptr(), wg.data_ptr(), wu.data_ptr(), out.data_ptr() + 16 * r0, 1) == 0
        _assert_tile(out, want, N, 30)
    M, N = 70, 256                                                     # many rows: padding only
    wg, wu = (binding.op_pack_tiled(dev(s, (N, 256), 0.1)) for s in (963, 964))
    am = binding.op_pack_tiled(dev(965, (M, 256)))
    out = torch.full((96 * N,), -7.0, dtype=torch.bfloat16, device="cuda")
    assert lib.mc_op_linear_swiglu(None, 1, M, N, 256, am.data_ptr(), wg.data_ptr(), wu.data_ptr(), out.data_ptr(), 1) == 0
    got = binding.tiled_to_rowmajor(out, 96, N)
    want = binding.tiled_to_rowmajor(binding.op_linear_swiglu(am, wg, wu, tiled_shape=(M, N, 256)), M, N)
    assert torch.equal(got[:M], want) and torch.all(got[M:] == -7)
    Hq, Hkv, pg = 8, 2, 64
    # a workgroup per candidate and KV head, merged states, one state, the generic kernel
    for hd, P, t, splits in ((64, 300, 20, 0), (64, 300, 20, 2), (128, 20, 0, 1), (96, 50, 9, 0)):
        for static in (False, True):
            kp, vp, _, _ = make_pools("bf16", -(-P // pg), Hkv, pg, hd, 966)
            ks, vs, _, _ = make_pools("bf16", 30, Hkv, pg, hd, 968)
            table = torch.arange(30, dtype=torch.int32, device="cuda").reshape(30, 1)
            q = dev(970, (30, Hq, hd))
            out = torch.full((64 * Hq * hd,), -7.0, dtype=torch.bfloat16, device="cuda")
            want = torch.full((30, Hq * hd), -7.0, dtype=torch.bfloat16, device="cuda")
            for r0, rows in _tile_calls(n):
                part = (q[r0:r0 + rows].contiguous(), kp, vp, ks, vs, table[r0:r0 + rows].contiguous(), P, t, pg, splits)
                binding.op_attention_decode(*part, out_tiled=True, out=out[8 * r0:], static_scratch=static)
                want[r0:r0 + rows] = binding.op_attention_decode(*part).reshape(rows, -1)
            _assert_tile(out, want, Hq * hd, 30)
            whole = binding.op_attention_decode(*part, out_tiled=True, static_scratch=static)
            assert not _padding_of(whole, rows, Hq * hd).any()


@pytest.mark.parametrize("Hq,hd,lens,kernel", [
    (8, 128, (300,), "pair"), (8, 64, (33,), "pair"), (8, 128, (1000, 70, 40), "pair"), (8, 64, (1000, 1000, 71), "pair"),
    (64, 128, (300,), "split"), (64, 64, (300,), "split"), (40, 128, (400, 1, 150), "split"), (64, 128, (1000, 65, 1000, 30), "whole"), (18, 64, (4000,) * 4, "rest")])
def test_prefill_attention_zeroes_the_rows_that_no_item_covers(Hq, hd, lens, kernel):
    """Padding rows, and rows between the items: in all forms (few and many workgroups, the last two with an output
    larger than the L2s)."""
    import torch
    Hkv, pg, P = 2, 64, 200
    items, row, holes = [], 0, []
    for n in lens:
        items += [[row + r, min(64, n - r), P - n % 100 + r, -1] for r in range(0, n, 64)]
        holes += list(range(row + n, row + n + 7))
        row += n + 7                                    # seven rows that nobody computes
    rows = row
    assert binding.op_attention_prefill_plan(len(items), Hq, Hkv, hd, pg, P + max(lens))[0] == kernel
    kp, vp, _, _ = make_pools("bf16", -(-(P + max(lens)) // pg), Hkv, pg, hd, 927)
    q = to_dev(rnd(928, (rows, Hq, hd)), "bf16")[0]
    it = torch.tensor(items, dtype=torch.int32, device="cuda")
    run = lambda tiled: binding.op_attention_prefill(q, it, kp, vp, None, None, None, P + max(lens), pg, out_tiled=tiled)  # noqa: E731
    _poison((rows + 31) // 32 * 32 * Hq * hd)
    out = run(True)
    plain = binding.tiled_to_rowmajor(out, rows, Hq * hd)
    assert not out.isnan().any() and not _padding_of(out, rows, Hq * hd).any() and not plain[holes].any()
    keep = [r for r in range(rows) if r not in set(holes)]
    assert torch.equal(plain[keep], run(False).reshape(rows, -1)[keep])


@pytest.mark.parametrize("Hq,Hkv,hd,P,rows", [(5, 1, 128, 64, 33), (40, 8, 128, 129, 70), (2, 2, 64, 1, 40), (3, 1, 64, 191, 64), (8, 2, 128, 2049, 5),
                                              (32, 8, 64, 2113, 64)])
def test_attention_prefill_pairs_of_heads(Hq, Hkv, hd, P, rows):
    """Workgroups of two heads with scoring and adding waves: odd and single heads per group, one page, odd and even page counts,
    steps that end among masked blocks.  A sequence alone (those workgroups) has the bits that it has among many (whole
    items), where a key that outgrows the reference stands in its suffix."""
    import torch
    n = -(-1100 // (2 * -(-Hq // Hkv // 2) * Hkv))
    pg, per, n_pre = 64, -(-rows // 64), -(-P // 64)
    g = torch.Generator(device="cuda")
    g.manual_seed(31 * P + Hq)
    normal = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)  # noqa: E731
    kp, vp = binding.kv_pages_pack(normal(n_pre, Hkv, pg, hd), normal(n_pre, Hkv, pg, hd))
    k = normal(n * per, Hkv, pg, hd)
    k[:, :, 3] *= 8
    ks, vs = binding.kv_pages_pack(k, normal(n * per, Hkv, pg, hd))
    table = torch.randperm(n * per, generator=g, device="cuda").to(torch.int32).reshape(n, per)
    q = normal(n * rows, Hq, hd) * 2

    def score(seqs):
        items = [[i * rows + j, min(64, rows - j), P + j, c] for i, c in enumerate(seqs) for j in range(0, rows, 64)]
        rq = torch.cat([q[c * rows: (c + 1) * rows] for c in seqs])
        out = binding.op_attention_prefill(rq, torch.tensor(items, dtype=torch.int32, device="cuda"), kp, vp, ks, vs, table, P, pg)
        return out.view(torch.int16).reshape(len(seqs), rows, Hq, hd)

    print("case: prefill pairs of heads", Hq, Hkv, hd, P, rows, n, flush=True)
    full = score(list(range(n)))
    assert not torch.isnan(full.view(torch.bfloat16)).any()
    for seqs in ([n // 2], [0, n - 1]):
        assert torch.equal(score(seqs), score(seqs)) and torch.equal(score(seqs), full[seqs])


@pytest.mark.parametrize("Hq,Hkv,hd", [(5, 1, 128), (10, 2, 64), (6, 1, 128), (2, 2, 64), (8, 4, 128)])
def test_attention_prefill_rest_heads_of_neighbouring_items(Hq, Hkv, hd):
    """One or two heads past a multiple of four: their workgroup takes up to four neighbouring items of one sequence.  Sequences of one to
    seven items, so that the groups of neighbours break at every place, short last items, two neighbours of one sequence that do not follow each
    other, prefix-only items at the end; each has the bits that it has alone (other kernels)."""
    import torch
    pg, P, G = 64, 200, Hq // Hkv
    lens = [64, 130, 5, 300, 64, 70, 448, 1, 193, 256]
    per = max(-(-n // 64) for n in lens)
    while binding.op_attention_prefill_plan(sum(-(-n // 64) for n in lens) + 4, Hq, Hkv, hd, pg, P, per)[0] != "rest":
        lens = lens + lens[1:]
    g = torch.Generator(device="cuda")
    g.manual_seed(77 + Hq + hd)
    normal = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)  # noqa: E731
    kp, vp = binding.kv_pages_pack(normal(-(-P // pg), Hkv, pg, hd), normal(-(-P // pg), Hkv, pg, hd))
    ks, vs = binding.kv_pages_pack(normal(len(lens) * per, Hkv, pg, hd), normal(len(lens) * per, Hkv, pg, hd))
    table = torch.randperm(len(lens) * per, generator=g, device="cuda").to(torch.int32).reshape(len(lens), per)
    items, row = [], 0
    for c, n in enumerate(lens):
        items += [[row + r, min(64, n - r), P + r, c] for r in range(0, n, 64)]
        row += n
    items += [[row, 64, 0, -1], [row + 64, 64, 64, -1], [row + 128, 8, P - 8, -1], [row + 136, 30, 10, -1]]
    row += 166
    items[4], items[5] = items[5], items[4]
    q = normal(row, Hq, hd)

    def run(some):
        print("case: prefill rest heads", Hq, Hkv, hd, len(some), flush=True)
        return binding.op_attention_prefill(q, torch.tensor(some, dtype=torch.int32, device="cuda"), kp, vp, ks, vs, table, P, pg).reshape(row, Hq, hd)

    full = run(items)
    assert not full.isnan().any()
    for i in list(range(0, 24)) + list(range(len(items) - 6, len(items))):
        r, n = items[i][:2]
        assert torch.equal(run([items[i]])[r: r + n], full[r: r + n]), (i, items[i])
