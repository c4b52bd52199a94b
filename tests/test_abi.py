"""The C ABI on the host (no GPU work): symbols and argument validation.

Every invalid call below is rejected by host-side validation before any HIP
call, so these run without a GPU.
"""
import ctypes

import pytest

from paper_2606_03928_amd import vase


@pytest.fixture(scope="module")
def lib():
    return vase.load()


def test_exports_every_declared_symbol(lib):
    names = vase.header_functions()
    assert set(names) == {"vase_workspace_bytes", "vase_score", "vase_score_ex", "vase_score_lse",
                          "vase_select", "vase_compact", "vase_decode_attn_lse", "vase_decode_step",
                          "vase_quantize", "vase_dequantize", "vase_compact_decode_ex",
                          "vase_decode_attn", "vase_compact_decode", "vase_dkv_projection",
                          "vase_dkv_score", "vase_status_str", "vase_version", "vase_score_map",
                          "vase_order_scores", "vase_compact_decode_map",
                          "vase_decode_step_noalloc"}
    for n in names:
        assert hasattr(lib, n), n


def test_version_and_status_strings(lib):
    assert vase.version() == (2, 0)
    for code in (0, -1, -2, -3, -4, -5):
        assert vase.status_str(code) != "unknown status"
    assert vase.status_str(-99) == "unknown status"


FAKE = ctypes.c_void_p(1 << 20)        # aligned, never dereferenced: calls fail validation first
MISALIGNED = ctypes.c_void_p((1 << 20) + 4)
UNALIGNED4 = ctypes.c_void_p((1 << 20) + 2)   # a status word must be 4-byte aligned


def _score(lib, **kw):
    a = dict(k=FAKE, v=FAKE, q=FAKE, dtype=0, n=4, K=256, B=32, d=128, G=2, w=16, pool=7,
             attn=FAKE, vr=FAKE, ws=FAKE, wsb=1 << 40, st=None)
    a.update(kw)
    return lib.vase_score(a["k"], a["v"], a["q"], a["dtype"], a["n"], a["K"], a["B"], a["d"],
                          a["G"], a["w"], a["pool"], a["attn"], a["vr"], a["ws"], a["wsb"], a["st"],
                          None)


@pytest.mark.parametrize("kw,code", [
    (dict(k=None), vase.ERR_INVALID_ARG),
    (dict(attn=None), vase.ERR_INVALID_ARG),
    (dict(dtype=7), vase.ERR_DTYPE),
    (dict(n=0), vase.ERR_INVALID_ARG),
    (dict(K=0), vase.ERR_INVALID_ARG),
    (dict(B=0), vase.ERR_INVALID_ARG),
    (dict(d=96), vase.ERR_INVALID_ARG),
    (dict(G=0), vase.ERR_INVALID_ARG),
    (dict(w=0), vase.ERR_INVALID_ARG),
    (dict(pool=4), vase.ERR_INVALID_ARG),
    (dict(pool=0), vase.ERR_INVALID_ARG),
    (dict(pool=257), vase.ERR_INVALID_ARG),
    (dict(q=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(ws=None), vase.ERR_WORKSPACE),
    (dict(wsb=16), vase.ERR_WORKSPACE),
    (dict(st=UNALIGNED4), vase.ERR_INVALID_ARG),
])
def test_score_validation(lib, kw, code):
    assert _score(lib, **kw) == code


def _score_ex(lib, kind, **kw):
    a = dict(k=FAKE, v=FAKE, q=FAKE, dtype=0, n=4, K=256, B=32, d=128, G=2, w=16, pool=7,
             attn=FAKE, vr=FAKE, ws=FAKE, wsb=1 << 40, st=None)
    a.update(kw)
    return lib.vase_score_ex(a["k"], a["v"], a["q"], a["dtype"], a["n"], a["K"], a["B"], a["d"],
                             a["G"], a["w"], a["pool"], kind, 1, 0, 0, a["attn"], a["vr"],
                             a["ws"], a["wsb"], a["st"], None)


@pytest.mark.parametrize("kind,kw,code", [
    (-1, {}, vase.ERR_INVALID_ARG),
    (5, {}, vase.ERR_INVALID_ARG),
    (vase.VALUE_RANGE, dict(vr=None), vase.ERR_INVALID_ARG),    # only VALUE_SKIP takes no vrange
    (vase.VALUE_SKIP, dict(attn=None), vase.ERR_INVALID_ARG),
    (vase.VALUE_L2, dict(v=None), vase.ERR_INVALID_ARG),
    (vase.VALUE_VAR, dict(vr=MISALIGNED), vase.ERR_INVALID_ARG),
    (vase.VALUE_RANDOM, dict(pool=2), vase.ERR_INVALID_ARG),
    (vase.VALUE_RANDOM, dict(dtype=9), vase.ERR_DTYPE),
    (vase.VALUE_L2, dict(ws=None), vase.ERR_WORKSPACE),
])
def test_score_ex_validation(lib, kind, kw, code):
    assert _score_ex(lib, kind, **kw) == code


def _select(lib, **kw):
    a = dict(attn=FAKE, vr=FAKE, n=4, base=0, K=256, B=32, Nv=16, seed=1, rnd=0, flags=0,
             src=FAKE, keys=None, st=None)
    a.update(kw)
    return lib.vase_select(a["attn"], a["vr"], a["n"], a["base"], a["K"], a["B"], a["Nv"],
                           a["seed"], a["rnd"], a["flags"], a["src"], a["keys"], a["st"], None)


@pytest.mark.parametrize("kw", [
    dict(attn=None), dict(src=None), dict(n=0), dict(K=0), dict(B=0), dict(Nv=-1),
    dict(Nv=225), dict(K=vase.MAX_K + 64, B=32), dict(flags=2), dict(keys=MISALIGNED),
    dict(st=UNALIGNED4),
])
def test_select_validation(lib, kw):
    assert _select(lib, **kw) == vase.ERR_INVALID_ARG


@pytest.mark.parametrize("kw,code", [
    (dict(k=None), vase.ERR_INVALID_ARG), (dict(src=None), vase.ERR_INVALID_ARG),
    (dict(dtype=3), vase.ERR_DTYPE), (dict(d=32), vase.ERR_INVALID_ARG),
    (dict(n=1, ws=None), vase.ERR_WORKSPACE),    # one instance uses the staging workspace
])
def test_compact_validation(lib, kw, code):
    a = dict(k=FAKE, v=FAKE, dtype=0, n=4, K=2048, B=128, d=128, src=FAKE, ws=FAKE, wsb=1 << 40)
    a.update(kw)
    rc = lib.vase_compact(a["k"], a["v"], a["dtype"], a["n"], a["K"], a["B"], a["d"], a["src"],
                          a["ws"], a["wsb"], None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(q=None), vase.ERR_INVALID_ARG), (dict(G=9), vase.ERR_INVALID_ARG),
    (dict(G=0), vase.ERR_INVALID_ARG), (dict(nv=0), vase.ERR_INVALID_ARG),
    (dict(nv=2048 + 128 + 1), vase.ERR_INVALID_ARG), (dict(dtype=5), vase.ERR_DTYPE),
    (dict(n=1, ws=None), vase.ERR_WORKSPACE),
])
def test_decode_validation(lib, kw, code):
    a = dict(k=FAKE, v=FAKE, q=FAKE, dtype=0, n=4, K=2048, B=128, d=128, G=4, nv=2048, out=FAKE,
             ws=FAKE, wsb=1 << 40)
    a.update(kw)
    rc = lib.vase_decode_attn(a["k"], a["v"], a["q"], a["dtype"], a["n"], a["K"], a["B"], a["d"],
                              a["G"], a["nv"], a["out"], a["ws"], a["wsb"], None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(q=None), vase.ERR_INVALID_ARG), (dict(np_=0), vase.ERR_INVALID_ARG),
    (dict(np_=2049), vase.ERR_INVALID_ARG),               # n_persist > n_valid
    (dict(lse=MISALIGNED), vase.ERR_INVALID_ARG), (dict(G=9), vase.ERR_INVALID_ARG),
    (dict(dtype=3), vase.ERR_DTYPE), (dict(n=1, ws=None), vase.ERR_WORKSPACE),
    (dict(n=1, wsb=64), vase.ERR_WORKSPACE),
])
def test_decode_lse_validation(lib, kw, code):
    a = dict(k=FAKE, v=FAKE, q=FAKE, dtype=0, n=4, K=2048, B=128, d=128, G=4, nv=2048, np_=2048,
             out=FAKE, lse=FAKE, ws=FAKE, wsb=1 << 40)
    a.update(kw)
    rc = lib.vase_decode_attn_lse(a["k"], a["v"], a["q"], a["dtype"], a["n"], a["K"], a["B"],
                                  a["d"], a["G"], a["nv"], a["np_"], a["out"], a["lse"], a["ws"],
                                  a["wsb"], None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(k_new=None), vase.ERR_INVALID_ARG), (dict(lse_win=None), vase.ERR_INVALID_ARG),
    (dict(q_win=None), vase.ERR_INVALID_ARG), (dict(pos=-1), vase.ERR_INVALID_ARG),
    (dict(pos=128), vase.ERR_INVALID_ARG), (dict(w=0), vase.ERR_INVALID_ARG),
    (dict(w=129), vase.ERR_INVALID_ARG),                  # window longer than the buffer
    (dict(G=9), vase.ERR_INVALID_ARG), (dict(v_new=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(dtype=4), vase.ERR_DTYPE), (dict(n=1, ws=None), vase.ERR_WORKSPACE),
])
def test_decode_step_validation(lib, kw, code):
    a = dict(k=FAKE, v=FAKE, k_new=FAKE, v_new=FAKE, q=FAKE, dtype=0, n=4, K=2048, B=128, d=128,
             G=4, w=128, pos=5, q_win=FAKE, lse_win=FAKE, out=FAKE, ws=FAKE, wsb=1 << 40)
    a.update(kw)
    rc = lib.vase_decode_step(a["k"], a["v"], a["k_new"], a["v_new"], a["q"], a["dtype"], a["n"],
                              a["K"], a["B"], a["d"], a["G"], a["w"], a["pos"], a["q_win"],
                              a["lse_win"], a["out"], a["ws"], a["wsb"], None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(lse=None), vase.ERR_INVALID_ARG), (dict(lse=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(kind=5), vase.ERR_INVALID_ARG), (dict(pool=8), vase.ERR_INVALID_ARG),
    (dict(dtype=2), vase.ERR_DTYPE), (dict(ws=None, n=4), vase.ERR_WORKSPACE),
])
def test_score_lse_validation(lib, kw, code):
    a = dict(k=FAKE, v=FAKE, q=FAKE, lse=FAKE, dtype=0, n=4, K=256, B=32, d=128, G=2, w=16, pool=7,
             kind=0, attn=FAKE, vr=FAKE, ws=FAKE, wsb=1 << 40)
    a.update(kw)
    rc = lib.vase_score_lse(a["k"], a["v"], a["q"], a["lse"], a["dtype"], a["n"], a["K"], a["B"],
                            a["d"], a["G"], a["w"], a["pool"], a["kind"], 1, 0, 0, a["attn"],
                            a["vr"], a["ws"], a["wsb"], None, None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(kind=vase.VALUE_RANDOM), vase.ERR_INVALID_ARG),   # nothing to carry for random scores
    (dict(kind=vase.VALUE_SKIP), vase.ERR_INVALID_ARG), (dict(kind=-1), vase.ERR_INVALID_ARG),
    (dict(vr=MISALIGNED), vase.ERR_INVALID_ARG), (dict(src=None), vase.ERR_INVALID_ARG),
    (dict(dtype=2), vase.ERR_DTYPE), (dict(n=1, ws=None), vase.ERR_WORKSPACE),
])
def test_compact_decode_ex_validation(lib, kw, code):
    a = dict(k=FAKE, v=FAKE, dtype=0, n=4, K=2048, B=128, d=128, src=FAKE, q=FAKE, G=4, out=FAKE,
             kind=vase.VALUE_RANGE, vr=FAKE, ws=FAKE, wsb=1 << 40)
    a.update(kw)
    rc = lib.vase_compact_decode_ex(a["k"], a["v"], a["dtype"], a["n"], a["K"], a["B"], a["d"],
                                    a["src"], a["q"], a["G"], a["out"], a["kind"], a["vr"], a["ws"],
                                    a["wsb"], None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(src=None), vase.ERR_INVALID_ARG), (dict(q=None), vase.ERR_INVALID_ARG),
    (dict(G=9), vase.ERR_INVALID_ARG), (dict(G=0), vase.ERR_INVALID_ARG),
    (dict(dtype=2), vase.ERR_DTYPE), (dict(d=96), vase.ERR_INVALID_ARG),
    (dict(out=ctypes.c_void_p((1 << 20) + 8)), vase.ERR_INVALID_ARG),
    (dict(n=1, ws=None), vase.ERR_WORKSPACE),    # one instance: the split two-step path
])
def test_compact_decode_validation(lib, kw, code):
    a = dict(k=FAKE, v=FAKE, dtype=0, n=4, K=2048, B=128, d=128, src=FAKE, q=FAKE, G=4, out=FAKE,
             ws=FAKE, wsb=1 << 40)
    a.update(kw)
    rc = lib.vase_compact_decode(a["k"], a["v"], a["dtype"], a["n"], a["K"], a["B"], a["d"],
                                 a["src"], a["q"], a["G"], a["out"], a["ws"], a["wsb"], None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(g=None), vase.ERR_INVALID_ARG), (dict(n=0), vase.ERR_INVALID_ARG),
    (dict(d=96), vase.ERR_INVALID_ARG), (dict(r=0), vase.ERR_INVALID_ARG),
    (dict(r=33), vase.ERR_INVALID_ARG), (dict(g=ctypes.c_void_p((1 << 20) + 4)), vase.ERR_INVALID_ARG),
])
def test_dkv_projection_validation(lib, kw, code):
    a = dict(n=4, base=0, d=128, r=20, seed=1, rnd=0, g=FAKE)
    a.update(kw)
    rc = lib.vase_dkv_projection(a["n"], a["base"], a["d"], a["r"], a["seed"], a["rnd"], a["g"], None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(k=None), vase.ERR_INVALID_ARG), (dict(g=None), vase.ERR_INVALID_ARG),
    (dict(dtype=7), vase.ERR_DTYPE), (dict(r=40), vase.ERR_INVALID_ARG),
    (dict(K=0), vase.ERR_INVALID_ARG), (dict(d=32), vase.ERR_INVALID_ARG),
    # decode logits: q_dec and the output together, 1 <= G <= 16, aligned, bf16
    (dict(k=None, qd=FAKE, dl=FAKE), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE, r=0), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE), vase.ERR_INVALID_ARG), (dict(dl=FAKE), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE, dl=FAKE, G=0), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE, dl=FAKE, G=17), vase.ERR_INVALID_ARG),
    (dict(qd=MISALIGNED, dl=FAKE), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE, dl=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE, dl=FAKE, dtype=1), vase.ERR_DTYPE),
])
def test_dkv_score_validation(lib, kw, code):
    a = dict(k=FAKE, v=FAKE, g=FAKE, dtype=0, n=4, K=2048, B=128, d=128, r=20, out=FAKE, qd=None,
             G=4, dl=None)
    a.update(kw)
    rc = lib.vase_dkv_score(a["k"], a["v"], a["g"], a["dtype"], a["n"], a["K"], a["B"], a["d"],
                            a["r"], a["out"], a["qd"], a["G"], a["dl"], None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(x=None), vase.ERR_INVALID_ARG), (dict(codes=None), vase.ERR_INVALID_ARG),
    (dict(bits=3), vase.ERR_INVALID_ARG), (dict(bits=16), vase.ERR_INVALID_ARG),
    (dict(group=16), vase.ERR_INVALID_ARG), (dict(d=64, group=128), vase.ERR_INVALID_ARG),
    (dict(Nv=-1), vase.ERR_INVALID_ARG), (dict(Nv=257), vase.ERR_INVALID_ARG),
    (dict(Nv=4, rng=None), vase.ERR_INVALID_ARG), (dict(Nv=4, hp=None), vase.ERR_INVALID_ARG),
    (dict(Nv=4, K=vase.MAX_K + 32), vase.ERR_INVALID_ARG), (dict(mse=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(dtype=5), vase.ERR_DTYPE), (dict(K=0), vase.ERR_INVALID_ARG),
])
def test_quantize_validation(lib, kw, code):
    a = dict(x=FAKE, dtype=0, n=4, K=256, B=32, d=128, bits=4, group=32, Nv=0, codes=FAKE,
             params=FAKE, rng=FAKE, mse=FAKE, hp=FAKE, idx=FAKE)
    a.update(kw)
    rc = lib.vase_quantize(a["x"], a["dtype"], a["n"], a["K"], a["B"], a["d"], a["bits"], a["group"],
                           a["Nv"], a["codes"], a["params"], a["rng"], a["mse"], a["hp"], a["idx"],
                           None)
    assert rc == code


@pytest.mark.parametrize("kw,code", [
    (dict(codes=None), vase.ERR_INVALID_ARG), (dict(out=None), vase.ERR_INVALID_ARG),
    (dict(bits=1), vase.ERR_INVALID_ARG), (dict(Nv=3, hp=None), vase.ERR_INVALID_ARG),
    (dict(params=MISALIGNED), vase.ERR_INVALID_ARG), (dict(dtype=9), vase.ERR_DTYPE),
])
def test_dequantize_validation(lib, kw, code):
    a = dict(codes=FAKE, params=FAKE, hp=FAKE, idx=FAKE, dtype=0, n=4, K=256, B=32, d=128, bits=4,
             group=32, Nv=0, out=FAKE)
    a.update(kw)
    rc = lib.vase_dequantize(a["codes"], a["params"], a["hp"], a["idx"], a["dtype"], a["n"], a["K"],
                             a["B"], a["d"], a["bits"], a["group"], a["Nv"], a["out"], None)
    assert rc == code


def test_workspace_sizes(lib):
    import torch
    # score needs partials unless one workgroup holds each instance (then it pools
    # by itself); select none; compact stages only when instances are split
    assert vase.workspace_bytes(vase.OP_SCORE, torch.bfloat16, 2304, 4096, 128, 128, 4, 128) == 0
    assert vase.workspace_bytes(vase.OP_SCORE, torch.bfloat16, 64, 4096, 128, 128, 4, 128) > 0
    assert vase.workspace_bytes(vase.OP_SCORE, torch.bfloat16, 2304, 8192, 256, 128, 5, 256) > 0
    assert vase.workspace_bytes(vase.OP_SCORE, torch.float32, 2304, 4096, 128, 128, 4, 128) > 0
    assert vase.workspace_bytes(vase.OP_SELECT, torch.bfloat16, 2304, 4096, 128, 128) == 0
    assert vase.workspace_bytes(vase.OP_COMPACT, torch.bfloat16, 2304, 4096, 128, 128) == 0
    assert vase.workspace_bytes(vase.OP_COMPACT, torch.bfloat16, 8, 2048, 128, 128) > 0
    # the fused call needs none when each instance fits one workgroup
    assert vase.workspace_bytes(vase.OP_COMPACT_DECODE, torch.bfloat16, 2304, 4096, 128, 128, 4) == 0
    assert vase.workspace_bytes(vase.OP_COMPACT_DECODE, torch.bfloat16, 8, 2048, 128, 128, 4) > 0
    assert vase.workspace_bytes(vase.OP_SCORE, torch.bfloat16, 0, 4096, 128, 128, 4, 128) == 0
    # decode: room for one more key split than n_valid = N alone needs (the
    # persistent boundary), so every (n_valid, n_persist) fits
    assert vase.workspace_bytes(vase.OP_DECODE, torch.bfloat16, 8, 2048, 128, 128, 4) > 0


def test_workspace_sizes_take_whole_numbers_only(lib):
    # also once the same size has been asked for as an int
    import ctypes
    import torch
    sizes = (2, 128, 32, 64, 2, 8)
    assert vase.workspace_bytes(vase.OP_SCORE, torch.float32, *sizes) > 0
    with pytest.raises(ctypes.ArgumentError):
        vase.workspace_bytes(vase.OP_SCORE, torch.float32, *map(float, sizes))


def _score_map(lib, **kw):
    a = dict(k=FAKE, v=FAKE, q=FAKE, lse=None, ord=FAKE, dtype=0, n=4, K=256, B=32, d=128, G=2,
             w=16, pool=7, kind=vase.VALUE_RANGE, attn=FAKE, vr=FAKE, qd=None, dl=None, ws=FAKE,
             wsb=1 << 40, st=None)
    a.update(kw)
    return lib.vase_score_map(a["k"], a["v"], a["q"], a["lse"], a["ord"], a["dtype"], a["n"],
                              a["K"], a["B"], a["d"], a["G"], a["w"], a["pool"], a["kind"], 1, 0, 0,
                              a["attn"], a["vr"], a["qd"], a["dl"], a["ws"], a["wsb"], a["st"], None)


@pytest.mark.parametrize("kw,code", [
    (dict(ord=None), vase.ERR_INVALID_ARG),
    (dict(ord=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(st=UNALIGNED4), vase.ERR_INVALID_ARG),
    (dict(K=vase.MAX_K + 32), vase.ERR_INVALID_ARG),
    (dict(k=None), vase.ERR_INVALID_ARG),
    (dict(pool=6), vase.ERR_INVALID_ARG),
    (dict(kind=7), vase.ERR_INVALID_ARG),
    (dict(lse=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(dtype=5), vase.ERR_DTYPE),
    (dict(ws=None), vase.ERR_WORKSPACE),       # the per-slot scores always need workspace
    (dict(n=64, K=4096, B=128, G=4, w=128, wsb=64 * 4096 * 4), vase.ERR_WORKSPACE),
    # decode logits: q_dec and the output go together, need the pass over every
    # key (no lse_win), at most 16 heads, bf16
    (dict(qd=FAKE), vase.ERR_INVALID_ARG),
    (dict(dl=FAKE), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE, dl=FAKE, lse=FAKE), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE, dl=FAKE, G=17), vase.ERR_INVALID_ARG),
    (dict(qd=MISALIGNED, dl=FAKE), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE, dl=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(qd=FAKE, dl=FAKE, dtype=1), vase.ERR_DTYPE),
])
def test_score_map_validation(lib, kw, code):
    assert _score_map(lib, **kw) == code


@pytest.mark.parametrize("kw", [
    dict(attn=None), dict(ord=None), dict(out=None), dict(vr=FAKE, vr_out=None), dict(n=0),
    dict(K=0), dict(K=vase.MAX_K + 1), dict(pool=2), dict(pool=257), dict(ord=MISALIGNED),
    dict(vr=MISALIGNED, vr_out=FAKE),
])
def test_order_scores_validation(lib, kw):
    a = dict(attn=FAKE, vr=None, ord=FAKE, n=4, K=256, pool=7, out=FAKE, vr_out=None)
    a.update(kw)
    rc = lib.vase_order_scores(a["attn"], a["vr"], a["ord"], a["n"], a["K"], a["pool"], a["out"],
                               a["vr_out"], None)
    assert rc == vase.ERR_INVALID_ARG


@pytest.mark.parametrize("kw,code", [
    (dict(k=None), vase.ERR_INVALID_ARG), (dict(src=None), vase.ERR_INVALID_ARG),
    (dict(ord=None), vase.ERR_INVALID_ARG), (dict(ord=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(q=None), vase.ERR_INVALID_ARG),                    # q and out go together
    (dict(out=None), vase.ERR_INVALID_ARG),
    (dict(q=None, out=None, vr=MISALIGNED), vase.ERR_INVALID_ARG),  # scores without the decode
    (dict(vr=FAKE, kind=vase.VALUE_RANDOM), vase.ERR_INVALID_ARG),
    (dict(G=0), vase.ERR_INVALID_ARG), (dict(G=9), vase.ERR_INVALID_ARG),
    (dict(K=vase.MAX_K + 64), vase.ERR_INVALID_ARG), (dict(K=16, B=32), vase.ERR_INVALID_ARG),
    (dict(dtype=2), vase.ERR_DTYPE), (dict(d=80), vase.ERR_INVALID_ARG),
    (dict(vin=FAKE), vase.ERR_INVALID_ARG),                  # scores in need scores out
    (dict(vin=MISALIGNED, vr=FAKE, K=16, B=32), vase.ERR_INVALID_ARG),
    # supplied decode logits: with the decode (q), G <= 8, aligned, bf16 only
    (dict(q=None, out=None, dl=FAKE), vase.ERR_INVALID_ARG),
    (dict(G=9, dl=FAKE), vase.ERR_INVALID_ARG),
    (dict(dl=MISALIGNED), vase.ERR_INVALID_ARG),
    (dict(dtype=1, dl=FAKE), vase.ERR_DTYPE),
])
def test_compact_decode_map_validation(lib, kw, code):
    a = dict(k=FAKE, v=FAKE, dtype=0, n=4, K=2048, B=128, d=128, src=FAKE, ord=FAKE, q=FAKE, G=4,
             out=FAKE, kind=vase.VALUE_RANGE, vin=None, vr=None, dl=None)
    a.update(kw)
    rc = lib.vase_compact_decode_map(a["k"], a["v"], a["dtype"], a["n"], a["K"], a["B"], a["d"],
                                     a["src"], a["ord"], a["q"], a["G"], a["out"], a["kind"],
                                     a["vin"], a["vr"], a["dl"], None)
    assert rc == code


def test_score_map_workspace(lib):
    import torch
    # one workgroup per instance pools through the map itself: no workspace
    assert vase.workspace_bytes(vase.OP_SCORE_MAP, torch.bfloat16, 2304, 4096, 128, 128, 4, 128) == 0
    # otherwise the score's own workspace plus the per-slot scores and value scores
    for dt, n in ((torch.bfloat16, 64), (torch.float32, 2304)):
        base = vase.workspace_bytes(vase.OP_SCORE, dt, n, 4096, 128, 128, 4, 128)
        got = vase.workspace_bytes(vase.OP_SCORE_MAP, dt, n, 4096, 128, 128, 4, 128)
        assert got >= base + 2 * n * 4096 * 4
    assert vase.workspace_bytes(vase.OP_SCORE_MAP, torch.bfloat16, 64, 4096, 128, 128, 0, 128) == 0


def test_header_constants_match_binding():
    """The binding's copies of the header's #define values are the header's."""
    import os
    import re
    hdr = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                            "include", "vase.h")).read()
    defs = dict(re.findall(r"#define (VASE_\w+) (-?\d+)", hdr))
    assert int(defs["VASE_MAX_K"]) == vase.MAX_K
    assert int(defs["VASE_DEC_LOGITS_LDS"]) == vase.DEC_LOGITS_LDS
    assert int(defs["VASE_OP_SCORE_MAP"]) == vase.OP_SCORE_MAP
    assert [int(defs[n]) for n in ("VASE_STATUS_ROW_NORM", "VASE_STATUS_VALUE_ROW",
                                   "VASE_STATUS_SELECT_ATTN", "VASE_STATUS_SELECT_VALUE")] == [
        vase.STATUS_ROW_NORM, vase.STATUS_VALUE_ROW, vase.STATUS_SELECT_ATTN,
        vase.STATUS_SELECT_VALUE]


def test_dec_logits_fit():
    # the Qwen3-8B shape's logits fit (G = 4, N = 4224: 67.6 KB + the queries);
    # the Qwen3-14B shape's do not (G = 5, N = 8448)
    assert vase.dec_logits_fit(4224, 128, 4)
    assert not vase.dec_logits_fit(8448, 128, 5)
    # the bound itself: G * ceil4(N) * 4 + G * d * 2 <= VASE_DEC_LOGITS_LDS
    n_max = (vase.DEC_LOGITS_LDS - 4 * 128 * 2) // 16
    assert vase.dec_logits_fit(n_max, 128, 4) and not vase.dec_logits_fit(n_max + 4, 128, 4)
