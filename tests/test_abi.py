"""Host-side checks of the C ABI: the library loads, exports every declared symbol, and its
sizing / validation code behaves (no GPU work is launched here)."""
import ctypes as C
import os
import re
import struct

import pytest

from paper_2601_05475_amd import binding, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__ as g
        g.build()
    return binding.load_library()


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "mc.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mc_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported_and_bound(lib):
    names = declared_symbols()
    assert {"mc_prefill_shared", "mc_decode_step", "mc_score_candidates", "mc_sample"} <= set(names)
    for n in names:
        assert hasattr(lib, n), f"{n} declared in mc.h but not exported"
        assert n in binding.SIGNATURES, f"{n} has no Python signature"
    assert set(binding.SIGNATURES) == set(names)


def test_model_and_session_sizes(lib):
    s = synth.TINY
    cfg = binding.make_config(s)
    nbytes = lib.mc_model_bytes(C.byref(cfg))
    d, F, V, hd = s.d_model, s.d_ffn, s.vocab, s.head_dim
    per_layer = 2 * d + (s.n_q_heads + 2 * s.n_kv_heads) * hd * d + d * s.n_q_heads * hd + 3 * F * d
    params = 2 * V * d + d + s.n_layers * per_layer
    assert params * 4 <= nbytes <= params * 4 + 256 * (4 + 7 * s.n_layers)
    p = binding.mc_session_params(128, 4, 16, 4, 0)
    sb = lib.mc_session_bytes(C.byref(cfg), C.byref(p))
    kv = 2 * s.n_layers * ((128 // 4) + 4 * 4) * s.n_kv_heads * hd * 4 * 4
    assert sb > kv
    # 8B shape, headline workload: weights ~16 GB, KV = 512 MiB prefix + 2 GiB suffix
    cfg8 = binding.make_config(synth.S8B)
    assert 16.0e9 < lib.mc_model_bytes(C.byref(cfg8)) < 16.2e9
    p8 = binding.mc_session_params(4096, 32, 512, 64, 4096)
    sb8 = lib.mc_session_bytes(C.byref(cfg8), C.byref(p8))
    assert sb8 > 2.5 * 2 ** 30 and sb8 < 6 * 2 ** 30
    # a smaller page pool shrinks the session by exactly the pages it leaves out (K and V, every layer)
    p8s = binding.mc_session_params(4096, 32, 512, 64, 4096, 64)
    page = 2 * 8 * 128 * 64 * 2 * 32
    assert sb8 - lib.mc_session_bytes(C.byref(cfg8), C.byref(p8s)) == (32 * 8 - 64) * page
    p8b = binding.mc_session_params(4096, 32, 512, 64, 4096, 10 ** 6)     # more than can be used: capped
    assert lib.mc_session_bytes(C.byref(cfg8), C.byref(p8b)) == sb8


def test_invalid_configs_are_rejected(lib):
    s = synth.TINY
    for field, bad in [("n_layers", 0), ("n_kv_heads", 3), ("head_dim", 7), ("dtype", 9), ("vocab", 0)]:
        cfg = binding.make_config(s)
        setattr(cfg, field, bad)
        assert lib.mc_model_bytes(C.byref(cfg)) == 0
        assert len(lib.mc_last_error()) > 0
    cfg = binding.make_config(s)
    for field, bad in [("page_tokens", 3), ("page_tokens", 256), ("max_cands", 0), ("max_suffix", 0), ("pool_pages", -1)]:
        p = binding.mc_session_params(128, 4, 16, 4, 0)
        setattr(p, field, bad)
        assert lib.mc_session_bytes(C.byref(cfg), C.byref(p)) == 0
    assert lib.mc_model_bytes(None) == 0
    # NULL handles are reported, not dereferenced
    assert lib.mc_session_sync(None) == -1
    assert lib.mc_decode_step(None, None, 1) == -1
    assert lib.mc_prefill_shared(None, None, 1) == -1
    h = C.c_void_p()
    assert lib.mc_model_create(C.byref(cfg), None, None, C.byref(h)) == -1
    assert lib.mc_op_linear(None, 0, 4, 4, 4, None, None, None, 1, 0) == -1
    assert lib.mc_op_tiled_bytes(33, 128) == 64 * 128 * 2 and lib.mc_op_tiled_bytes(33, 100) == 0
    assert lib.mc_op_linear_splits(1, 32, 6144, 4096, 1) >= 1
    assert lib.mc_op_sample(None, 0, 10, None, 0, 1.0, 5, None, None, None) == -1
    # the fused many-row layers: bad arguments and shapes they do not cover are refused on the host
    fake = C.c_void_p(256)                     # never dereferenced: the checks come first
    assert lib.mc_op_linear_accumulate(None, 4096, 4096, 4096, None, None, None) == -1
    assert lib.mc_op_linear_accumulate(None, 0, 4096, 4096, fake, fake, fake) == -1
    assert lib.mc_op_linear_accumulate(None, 64, 4096, 4096, fake, fake, fake) == -5       # few rows: the weight-streaming path
    assert lib.mc_op_linear_accumulate(None, 8192, 4000, 4096, fake, fake, fake) == -5     # N not a multiple of 128
    assert lib.mc_op_linear_accumulate(None, 8192, 4096, 4000, fake, fake, fake) == -5     # K not a multiple of 256
    args = [fake] * 9
    assert lib.mc_op_linear_qkv_rope(None, 32, 32, 8, 128, 64, 4096, 5e5, 100, *([None] * 9)) == -1
    assert lib.mc_op_linear_qkv_rope(None, 32, 32, 8, 126, 64, 4096, 5e5, 100, *args) == -1   # head_dim % 4
    assert lib.mc_op_linear_qkv_rope(None, 32, 32, 8, 128, 64, 4096, -1.0, 100, *args) == -1
    out = (C.c_int32 * 9)()
    assert lib.mc_op_attention_decode_plan(32, 32, 8, 128, 64, 4096, 1, 0, out) == 0 and out[2] >= 1
    assert lib.mc_op_attention_decode_plan(32, 32, 8, 128, 64, 0, 0, 0, out) == -1           # no keys
    assert lib.mc_op_attention_decode_plan(32, 32, 7, 128, 64, 4096, 1, 0, out) == -1        # heads do not divide
    assert lib.mc_op_attention_decode_plan(32, 32, 8, 96, 64, 4096, 1, 0, out) == -5         # head_dim not covered
    assert lib.mc_op_attention_decode_plan(32, 32, 8, 128, 16, 4096, 1, 0, out) == -5        # page size not covered


def test_decode_attention_plan_covers_every_block_and_fits_its_workspace(lib):
    """Host logic of the decode-attention launcher: for a sweep of shapes the key splits cover
    every 32-key block exactly once, no split is empty, the partial states fit the workspace the
    library asks for, and the prefix ids of one split are a multiple of 8 apart."""
    import itertools
    shapes = [(32, 32, 8, 128), (64, 40, 8, 128), (16, 32, 8, 64), (1, 4, 4, 64), (5, 12, 2, 128), (33, 4, 1, 64)]
    lens = [0, 1, 31, 32, 33, 64, 65, 200, 512, 1000, 4096, 16384, 40000]
    for (B, Hq, Hkv, hd), P, t, S in itertools.product(shapes, lens, [0, 1, 63, 64, 65, 512, 1024, 3000], [0, 1, 7, 64, 5000]):
        if P + t == 0:
            continue
        p = binding.op_attention_decode_plan(B, Hq, Hkv, hd, 64, P, t, S)
        G = Hq // Hkv
        nb_p, nb_s = -(-P // 32), -(-t // 32)
        if P:
            assert p["splits"] >= 1 and p["splits"] * p["blocks_per_split"] >= nb_p
            assert (p["splits"] - 1) * p["blocks_per_split"] < nb_p
            row_blocks = -(-B * G // 32)
            assert p["rb_per_item"] == (4 if row_blocks >= 8 else 1)
            assert p["prefix_stride"] % 8 == 0 and p["prefix_stride"] >= Hkv * p["splits"]
            assert p["prefix_items"] == p["prefix_stride"] * -(-row_blocks // p["rb_per_item"])
        else:
            assert p["prefix_items"] == 0
        if t:
            assert 1 <= p["suffix_splits"] <= 8 and p["suffix_splits"] * p["suffix_bps"] >= nb_s
            assert (p["suffix_splits"] - 1) * p["suffix_bps"] < nb_s
            assert p["suffix_items"] == B * Hkv * p["suffix_splits"]
        else:
            assert p["suffix_items"] == 0
        assert p["n_parts"] == (p["splits"] if P else 0) + (p["suffix_splits"] if t else 0) <= 1024 or P > 100000
        ws = lib.mc_op_attention_decode_ws(B, Hq, Hkv, hd, P, t, 64)
        assert p["n_parts"] * B * Hq * (hd + 2) * 4 <= ws, (B, Hq, Hkv, hd, P, t, S, p, ws)


def test_tiled_entry_points_refuse_what_the_plain_ones_refuse(lib):
    """Host checks, pointers never followed: NULL pointers, fp32 and widths without the layout, a workspace too small."""
    p = C.c_void_p(256)
    assert lib.mc_op_add_rmsnorm_tiled(None, 1, 3, 64, None, None, 0, p, 1e-6, p) == -1
    assert lib.mc_op_add_rmsnorm_tiled(None, 0, 3, 64, p, None, 0, p, 1e-6, p) == -5
    assert lib.mc_op_add_rmsnorm_tiled(None, 1, 3, 96, p, None, 0, p, 1e-6, p) == -5
    assert lib.mc_op_add_rmsnorm(None, 1, 3, 64, p, None, 0, p, 1e-6, p, 2) == -1
    assert lib.mc_op_linear_swiglu_tiled(None, 1, 3, 128, 256, p, p, None, p) == -1
    assert lib.mc_op_linear_swiglu_tiled(None, 0, 3, 128, 256, p, p, p, p) == -5
    assert lib.mc_op_linear_swiglu_tiled(None, 1, 3, 100, 256, p, p, p, p) == -5
    assert lib.mc_op_linear_swiglu(None, 1, 3, 128, 256, p, p, p, p, 2) == -1
    sizes = (4, 8, 2, 64, 64, 100, 0)
    tail = (p, p, p, None, None, None, 0, None, 0)
    assert lib.mc_op_attention_decode_tiled(None, 1, *sizes, *tail, p, 16, p) == -1
    assert lib.mc_op_attention_decode_tiled(None, 0, *sizes, *tail, p, 1 << 30, p) == -5
    assert lib.mc_op_attention_decode_tiled(None, 1, *sizes, *tail, p, 1 << 30, None) == -1
    assert lib.mc_op_attention_decode(None, 1, *sizes, *tail, p, 1 << 30, p, 2) == -1


@pytest.mark.parametrize("B,Hq,Hkv,P", [(64, 40, 8, 16384), (57, 40, 8, 9000), (64, 32, 8, 4096), (64, 32, 4, 2048)])
def test_decode_attention_prefix_splits_do_not_follow_the_suffixes(B, Hq, Hkv, P):
    """Many query rows: the plan tells the splits of a launch whose candidates differ in length too (it is not told of them), and
    a rollout's prefix splits stay what they are while its suffixes grow."""
    assert len({binding.op_attention_decode_plan(B, Hq, Hkv, 128, 64, P, t, 0)["splits"] for t in (1, 64, 200, 353, 512, 1024, 4096)}) == 1


def test_gemm_plan_takes_96_rows_only_for_a_third_more_workgroups(lib):
    """Host logic of the many-row GEMM: one round of workgroups where a listed shape can have it, and the 96-row form in
    place of 128 x 64 only over a long K and where it has at least 4/3 of the workgroups (with 1.17 and 1.20 of
    them it was slower)."""
    for N, K in ((2048, 12288), (3072, 16384), (4096, 14336), (4096, 4096), (5120, 27648), (2048, 8192)):
        taken = 0
        for M in range(65, 1200):
            rows, cols, groups = binding.op_gemm_plan(M, N, K)
            assert groups == -(-M // rows) * (N // cols)
            by_128 = -(-M // 128) * (N // 64)
            if rows == 96:
                taken += 1
                assert cols == 64 and K >= 12288 and 3 * groups >= 4 * by_128 and groups <= 256, (M, N, K)
            assert groups <= 256 or -(-M // 128) * (N // 128) > 256, (M, N, K)
        assert (taken > 0) == (K >= 12288), (N, K)
    assert binding.op_gemm_plan(641, 2048, 12288) == (128, 64, 192)
    assert binding.op_gemm_plan(600, 2048, 12288) == (96, 64, 224)
    out = (C.c_int32 * 3)()
    assert lib.mc_op_gemm_plan(64, 4096, 4096, 0, out) == -5 and lib.mc_op_gemm_plan(65, 4000, 4096, 0, out) == -5
    assert lib.mc_op_gemm_plan(65, 4096, 4000, 1, out) == -5 and lib.mc_op_gemm_plan(0, 4096, 4096, 0, out) == -1
    assert lib.mc_op_gemm_plan(65, 4096, 4096, 2, out) == -1 and lib.mc_op_gemm_plan(65, 4096, 4096, 0, None) == -1


@pytest.mark.parametrize("M,N,K,form", [
    (900, 4096, 14336, (128, 128)), (1000, 4096, 14336, (128, 128)), (768, 5120, 27648, (128, 128)), (900, 4096, 8192, (128, 128)), (2000, 2048, 8192, (128, 128)),
    (900, 4096, 4096, (128, 128)), (400, 6144, 4096, (128, 128)), (400, 7168, 5120, (128, 128)), (959, 4096, 4096, (128, 128)),
    (960, 4096, 4096, (256, 64)), (1000, 4096, 4096, (256, 64)), (450, 6144, 4096, (256, 64)), (512, 7168, 5120, (256, 64)), (768, 5120, 5120, (256, 64)),
    (500, 5120, 5120, (192, 64)), (600, 4096, 14336, (192, 64)), (1000, 3072, 2048, (128, 128))])
def test_gemm_plan_takes_256_x_64_only_with_full_row_tiles_and_a_short_k(lib, M, N, K, form):
    """Weights in bursts by 256 x 64 lose where the last row tile is not full to three quarters (4096 x 14336, 900 rows 136 us by it, 114 by
    128 x 128) and over a K above 5120."""
    assert binding.op_gemm_plan(M, N, K)[:2] == form


@pytest.mark.parametrize("n,Hq,Hkv,hd,keys,stride,form", [
    # one round of workgroups of scoring and adding waves: always
    (5, 32, 8, 128, 4396, 0, "pair"), (8, 32, 8, 64, 65, 1, "pair"), (16, 16, 8, 128, 100, 2, "pair"),
    # a second round, one sequence (keys: its rows among them): against two waves per head from a length on, against whole items always
    (10, 32, 8, 128, 767, 0, "split"), (10, 32, 8, 128, 768, 0, "pair"), (16, 32, 8, 128, 1256, 0, "pair"), (5, 64, 8, 128, 1324, 0, "split"),
    (5, 64, 8, 128, 2348, 0, "pair"), (7, 40, 8, 128, 464, 0, "split"), (7, 48, 8, 64, 464, 0, "split"), (8, 48, 8, 64, 564, 0, "pair"),
    (10, 40, 8, 128, 664, 0, "pair"), (17, 8, 8, 128, 1100, 0, "pair"),
    # a second round, several sequences
    (16, 32, 8, 128, 3071, 1, "split"), (16, 32, 8, 128, 3072, 1, "pair"), (16, 32, 8, 64, 2047, 1, "split"), (16, 32, 8, 64, 2048, 1, "pair"),
    (32, 16, 8, 128, 2047, 1, "whole"), (32, 16, 8, 128, 2048, 1, "pair"),
    # more workgroups
    (17, 32, 8, 128, 4096, 0, "whole"), (128, 32, 8, 128, 4096, 16, "whole"), (33, 32, 8, 64, 9000, 1, "whole")])
def test_prefill_attention_takes_a_second_round_where_it_is_faster(lib, n, Hq, Hkv, hd, keys, stride, form):
    """Host logic of the prefill attention launcher at both sides of its lines (300 rows of 64 / 8 heads after 256 keys: 20.1 us by scoring and
    adding waves, 18.0 by two waves per head)."""
    kernel, groups = binding.op_attention_prefill_plan(n, Hq, Hkv, hd, 64, keys, stride)
    G = Hq // Hkv
    assert kernel == form
    assert groups == n * Hkv * {"whole": -(-G // 4), "split": 2 * -(-G // 4), "pair": 2 * -(-G // 2)}[kernel]


@pytest.mark.parametrize("n,Hq,Hkv,hd,keys,stride,form", [
    (32, 40, 8, 128, 4096, 1, "rest"), (32, 40, 8, 128, 4096, 2, "rest"), (32, 40, 8, 128, 4096, 4, "whole"), (40, 40, 8, 128, 4096, 5, "rest"),
    (24, 40, 8, 128, 4096, 4, "rest"), (128, 40, 8, 128, 4096, 16, "rest"), (16, 40, 8, 128, 300, 1, "whole"),
    (64, 16, 8, 128, 999, 1, "whole"), (64, 16, 8, 128, 1000, 1, "rest"), (64, 16, 8, 64, 64, 4, "rest"), (128, 8, 8, 128, 64, 16, "rest"),
    (64, 8, 8, 64, 3000, 4, "whole"), (65, 8, 8, 64, 3000, 4, "rest"), (65, 8, 8, 64, 300, 1, "whole"), (128, 32, 8, 128, 4096, 16, "whole"), (128, 56, 8, 128, 64, 1, "whole")])
def test_prefill_attention_takes_neighbouring_items_where_it_is_faster(lib, n, Hq, Hkv, hd, keys, stride, form):
    """Whole items, the heads past a multiple of four: at both sides of the lines (33 x 64 rows of 8 / 8 heads of 64 after 3000 keys: 62 us by
    neighbours, 56 by an item each; 64 x 64 rows of 16 / 8 heads of 128 after 64 keys 25.7 / 21.0)."""
    assert binding.op_attention_prefill_plan(n, Hq, Hkv, hd, 64, keys, stride)[0] == form


def test_prefill_attention_plan_refuses_what_the_launch_refuses(lib):
    out = (C.c_int32 * 2)()
    plan = lib.mc_op_attention_prefill_plan
    assert plan(5, 32, 8, 128, 64, 300, 0, out) == 0 and plan(5, 32, 8, 128, 64, 300, 0, None) == -1
    for bad in ((0, 32, 8, 128, 64, 300, 0), (5, 32, 7, 128, 64, 300, 0), (5, 32, 8, 128, 64, 0, 0), (5, 32, 8, 128, 64, 300, -1)):
        assert plan(*bad, out) == -1, bad
    assert plan(5, 32, 8, 96, 64, 300, 0, out) == -5 and plan(5, 32, 8, 128, 32, 300, 0, out) == -5


@pytest.mark.parametrize("rows,K,calls", [(1, 64, 1), (32, 2048, 1), (33, 4096, 1), (55, 5120, 1), (64, 128, 1), (300, 4096, 1),
                                          (300, 14336, 3)])
def test_tiled_outputs_cost_one_torch_call_and_have_zero_padding(rows, K, calls):
    """The buffer of a tiled output: its size, zeros in the padding rows where the operation does not write them, and
    then no more torch calls than a plain zeroed tensor takes unless it is large; one call where it does."""
    import torch
    from torch.utils._python_dispatch import TorchDispatchMode

    class Count(TorchDispatchMode):
        seen = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            Count.seen += 1
            return func(*args, **(kwargs or {}))

    with Count():
        out = binding._tiled_out(rows, K, torch.bfloat16, "cpu")
    assert Count.seen == calls
    with Count():
        whole = binding._tiled_empty(rows, K, torch.bfloat16, "cpu")
    assert Count.seen == calls + 1 and whole.dtype == out.dtype and whole.shape == out.shape
    assert out.dtype == torch.bfloat16 and out.numel() * 2 == binding.load_library().mc_op_tiled_bytes(rows, K)
    if rows % 32:
        assert not binding.tiled_to_rowmajor(out, (rows + 31) // 32 * 32, K)[rows:].any()


def _vgprs_allocated():
    """{kernel name: vector registers that a wave of it is given}, from the kernel descriptors of the library."""
    blob, out, at = open(binding.LIB_PATH, "rb").read(), {}, 0
    while (at := blob.find(b"\x7fELF\x02\x01\x01\x40", at + 1)) > 0:           # the device code objects inside
        shoff, = struct.unpack_from("<Q", blob, at + 40)
        shsize, shnum = struct.unpack_from("<HH", blob, at + 58)
        heads = [struct.unpack_from("<IIQQQQIIQQ", blob, at + shoff + i * shsize) for i in range(shnum)]
        for _, kind, _, _, off, size, link, _, _, entry in heads:
            if kind != 11:                                                          # dynamic symbols
                continue
            names = at + heads[link][4]
            for sym in range(at + off, at + off + size, entry):
                name, _, _, sec, value, _ = struct.unpack_from("<IBBHQQ", blob, sym)
                text = blob[names + name: blob.index(b"\0", names + name)].decode()
                if text.endswith(".kd") and sec < shnum:
                    kd = at + heads[sec][4] + value - heads[sec][3]
                    out[text[:-3]] = ((struct.unpack_from("<I", blob, kd + 48)[0] & 63) + 1) * 8
    return out


def test_prefill_attention_leaves_room_for_a_second_workgroup(lib):
    """512 registers per lane and SIMD: at head_dim 64 two workgroups of eight waves share a compute unit, and
    a bound on the waves per SIMD must not take that from them."""
    regs = {k: v for k, v in _vgprs_allocated().items() if "prefill_attention_kernelILi64E" in k}
    assert regs
    for name, n in regs.items():
        assert 512 // n >= 4, (name, n)


def test_bench_refuses_more_than_one_gpu_and_bad_step_counts():
    """bench.py is a one-GPU program: --gpus N > 1 ends with a message and a non-zero status before
    anything touches a device; so do step counts outside the workload."""
    import subprocess
    import sys
    bench = os.path.join(ROOT, "bench.py")
    r = subprocess.run([sys.executable, bench, "--gpus", "2"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 2 and "one GPU" in r.stderr and r.stdout.strip() == ""
    r = subprocess.run([sys.executable, bench, "--gpus", "0"], capture_output=True, text=True, timeout=300)
    assert r.returncode != 0 and r.stdout.strip() == ""
