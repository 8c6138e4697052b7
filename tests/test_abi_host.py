"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every symbol the header declares, and every argument error is reported before
anything could be launched."""
import ctypes as C
import os
import re
import struct

import pytest

from paper_2602_07899_amd import tlq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "tlq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(tlq_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = _declared_symbols()
    assert len(names) >= 15
    l = tlq.lib()
    for n in names:
        assert hasattr(l, n), f"{n} declared in tlq.h but not exported"
    assert set(names) == set(tlq.EXPORTS), "binding and header disagree"
    assert tlq.version() == 100
    assert tlq.status_string(tlq.OK) == "ok"
    assert "workspace" in tlq.status_string(tlq.ERR_WORKSPACE)


def test_params_struct_layout():
    assert C.sizeof(tlq.Params) == 32
    p = tlq.params()
    assert p.struct_size == 32 and p.bits == 4 and p.group == 128


FAKE = C.c_void_p(0x1000)        # aligned, never dereferenced: validation fails first
ODD = C.c_void_p(0x1004)


def _search(p, X=FAKE, n=256, ci=512, ldx=512, W=FAKE, co=512, ldw=512, Y=FAKE, ldy=512, w=FAKE,
            al=FAKE, na=20, best=FAKE, idx=FAKE, losses=FAKE, ws=FAKE, wsb=1 << 40):
    return tlq.lib().tlq_scale_search(X, n, ci, ldx, W, co, ldw, Y, ldy, w, al, na, C.byref(p), None,
                                      best, idx, losses, None, ws, wsb, None)


def test_scale_search_rejects_bad_arguments():
    p = tlq.params()
    assert _search(p, X=None) == tlq.ERR_NULL
    assert _search(p, losses=None) == tlq.ERR_NULL
    assert _search(p, n=0) == tlq.ERR_SHAPE
    assert _search(p, ldx=256) == tlq.ERR_SHAPE               # stride smaller than row
    assert _search(p, ci=520, ldx=520, ldw=520) == tlq.ERR_SHAPE   # not a multiple of group
    assert _search(p, ci=508, ldx=512, ldw=512) == tlq.ERR_SHAPE   # not a multiple of 8
    assert _search(p, na=0) == tlq.ERR_SHAPE
    assert _search(p, na=tlq.MAX_ALPHA + 1) == tlq.ERR_SHAPE
    assert _search(p, X=ODD) == tlq.ERR_ALIGN
    assert _search(p, ldy=516) == tlq.ERR_ALIGN
    assert _search(p, ws=None) == tlq.ERR_WORKSPACE
    assert _search(p, wsb=1024) == tlq.ERR_WORKSPACE
    for field, bad in [("bits", 1), ("bits", 9), ("group", 100), ("symmetric", 2), ("act_bits", 1), ("act_bits", 9),
                       ("xstat_kind", 2), ("x_dtype", tlq.F32), ("yref_dtype", 3), ("struct_size", 28)]:
        q = tlq.params()
        setattr(q, field, bad)
        assert _search(q) == tlq.ERR_UNSUPPORTED, field


def test_other_entry_points_reject_bad_arguments():
    l = tlq.lib()
    p = tlq.params()
    bp = C.byref(p)
    assert l.tlq_x_stat(None, 4, 8, 8, bp, FAKE, FAKE, 1 << 30, None) == tlq.ERR_NULL
    assert l.tlq_x_stat(FAKE, 4, 12, 16, bp, FAKE, FAKE, 1 << 30, None) == tlq.ERR_SHAPE
    assert l.tlq_x_stat(FAKE, 4, 8, 8, bp, FAKE, None, 0, None) == tlq.ERR_WORKSPACE
    assert l.tlq_scale_table(FAKE, 8, None, 4, FAKE, None) == tlq.ERR_NULL
    assert l.tlq_scale_table(FAKE, 8, FAKE, 0, FAKE, None) == tlq.ERR_SHAPE
    assert l.tlq_fake_quant(None, 4, 128, 128, None, bp, None, None, None, None, 0, None) == tlq.ERR_NULL
    assert l.tlq_fake_quant(FAKE, 4, 192, 192, None, bp, None, None, None, None, 0, None) == tlq.ERR_SHAPE
    assert l.tlq_fake_quant(ODD, 4, 128, 128, None, bp, None, None, None, None, 0, None) == tlq.ERR_ALIGN
    assert l.tlq_fake_quant(FAKE, 4, 128, 128, None, bp, None, None, None, FAKE, 64, None) == tlq.ERR_SHAPE
    assert l.tlq_weighted_layer_err(FAKE, 4, 128, 128, FAKE, 4, 128, None, FAKE, 8, None, bp, FAKE,
                                    None, FAKE, 1 << 30, None) == tlq.ERR_NULL
    assert l.tlq_weighted_layer_err(FAKE, 4, 128, 128, FAKE, 4, 128, None, FAKE, 8, FAKE, bp, FAKE,
                                    None, FAKE, 16, None) == tlq.ERR_WORKSPACE
    assert l.tlq_ref_output(FAKE, 4, 128, 128, FAKE, 4, 128, None, 8, bp, None) == tlq.ERR_NULL
    assert l.tlq_ref_output(FAKE, 4, 128, 128, FAKE, 4, 128, FAKE, 2, bp, None) == tlq.ERR_SHAPE
    assert l.tlq_apply_best(FAKE, 4, 128, 128, FAKE, 4, 128, None, bp, FAKE, 8, FAKE, 1 << 30,
                            None) == tlq.ERR_NULL
    assert l.tlq_apply_best(FAKE, 4, 128, 128, FAKE, 4, 128, FAKE, bp, FAKE, 8, FAKE, 8,
                            None) == tlq.ERR_WORKSPACE
    assert l.tlq_profile_get(99, None, 0, None, None, None) == tlq.ERR_SHAPE
    assert l.tlq_token_importance(None, 2, 4, 8, 8, 0, bp, FAKE, FAKE, 1 << 20, None) == tlq.ERR_NULL
    assert l.tlq_token_importance(FAKE, 2, 4, 8, 4, 0, bp, FAKE, FAKE, 1 << 20, None) == tlq.ERR_SHAPE
    assert l.tlq_token_importance(FAKE, 2, 4, 8, 8, 0, bp, FAKE, None, 0, None) == tlq.ERR_WORKSPACE
    assert l.tlq_topk_mask(FAKE, 4, 5, FAKE, None) == tlq.ERR_SHAPE
    assert l.tlq_topk_mask(FAKE, 1 << 20, 5, FAKE, None) == tlq.ERR_UNSUPPORTED
    assert l.tlq_x_stat_masked(FAKE, 4, 8, 8, None, 2, bp, FAKE, FAKE, 1 << 20, None) == tlq.ERR_NULL
    assert l.tlq_x_stat_masked(FAKE, 4, 8, 8, FAKE, 0, bp, FAKE, FAKE, 1 << 20, None) == tlq.ERR_SHAPE
    assert l.tlq_rmsnorm_mul(None, 4, 8, 8, None, 0, None, None, 0, 0, bp, FAKE, 8, None) == tlq.ERR_NULL
    assert l.tlq_rmsnorm_mul(FAKE, 4, 8, 8, None, 0, None, None, 0, 0, bp, FAKE, 4, None) == tlq.ERR_SHAPE
    assert l.tlq_rmsnorm_mul(FAKE, 4, 8, 8, None, 0, None, None, 4, 2, bp, FAKE, 8, None) == tlq.ERR_SHAPE
    att = lambda **k: l.tlq_causal_attention(k.get("Q", FAKE), k.get("ld", 256), FAKE, 256, FAKE, 256, k.get("n", 64),
                                             k.get("heads", 2), k.get("dh", 128), k.get("seq", 32), bp,
                                             k.get("out", FAKE), k.get("ldo", 256), None)
    assert att(Q=None) == tlq.ERR_NULL and att(out=None) == tlq.ERR_NULL
    assert att(dh=64) == tlq.ERR_UNSUPPORTED
    assert att(seq=48) == tlq.ERR_SHAPE            # 64 tokens are not whole samples of 48
    assert att(seq=0) == tlq.ERR_SHAPE and att(heads=0) == tlq.ERR_SHAPE and att(n=0) == tlq.ERR_SHAPE
    assert att(ld=128) == tlq.ERR_SHAPE and att(ldo=200) == tlq.ERR_SHAPE      # narrower than heads*128
    assert att(Q=ODD) == tlq.ERR_ALIGN and att(ld=260) == tlq.ERR_ALIGN
    for fn in (l.tlq_silu_mul, l.tlq_residual_add):
        assert fn(None, 8, FAKE, 8, 4, 8, bp, FAKE, 8, None) == tlq.ERR_NULL
        assert fn(FAKE, 8, FAKE, 8, 4, 8, bp, None, 8, None) == tlq.ERR_NULL
        assert fn(FAKE, 16, FAKE, 16, 4, 12, bp, FAKE, 16, None) == tlq.ERR_SHAPE   # width not a multiple of 8
        assert fn(FAKE, 8, FAKE, 4, 4, 8, bp, FAKE, 8, None) == tlq.ERR_SHAPE
        assert fn(FAKE, 8, FAKE, 8, 0, 8, bp, FAKE, 8, None) == tlq.ERR_SHAPE
        assert fn(ODD, 8, FAKE, 8, 4, 8, bp, FAKE, 8, None) == tlq.ERR_ALIGN


def test_workspace_queries():
    p = tlq.params()
    q = tlq.scale_search_workspace_bytes
    assert q(0, 512, 512, 20, p) == 0 and q(256, 512, 512, 0, p) == 0
    small, big = q(256, 512, 512, 20, p), q(10240, 4096, 4096, 20, p)
    assert small % 256 == 0 and small >= 20 * 512 * 512 * 2
    assert big >= 20 * 4096 * 4096 * 2 and big < 20 * 4096 * 4096 * 2 + (64 << 20)
    assert q(256, 512, 512, 10, p) < small
    bad = tlq.params(bits=1)
    assert q(256, 512, 512, 20, bad) == 0
    assert tlq.x_stat_workspace_bytes(256, 512) >= 2 * 512 * 8
    assert tlq.apply_best_workspace_bytes(256, 512, 512, p) >= 512 * 512 * 2
    pb = tlq.params(x_dtype=tlq.BF16)
    assert (tlq.apply_best_workspace_bytes(256, 512, 512, pb)
            >= tlq.apply_best_workspace_bytes(256, 512, 512, p) + 256 * 512 * 2)
    assert q(256, 512, 512, 20, pb) >= small + 256 * 512 * 2
    assert tlq.weighted_layer_err_workspace_bytes(256, 512, 512, p) >= 512 * 512 * 2


def _launch_tiles(n_tok, c_out, n_cand, tokens):
    """Tiles of a launch whose tiles hold `tokens` tokens (128 x 128 outputs, 256 outputs otherwise)."""
    return n_cand * -(-n_tok // tokens) * -(-c_out // (128 if tokens == 128 else 256))


# the last number is the token count of the tiles of the launch that the library makes
@pytest.mark.parametrize("shape", [
    (256, 512, 512, 20, 128),            # small case: one tile column
    (10240, 4096, 4096, 20, 320),        # 7B attention linear: one token chunk
    (10240, 4096, 11008, 20, 320),       # 43 tile rows: last patch row has 3 (3 x 10 patches)
    (10240, 11008, 4096, 20, 320),       # deep linear: several token chunks
    (40960, 4096, 11008, 20, 320),       # 128 tile columns in chunks of 4 patches
    (153600, 5120, 13824, 20, 320),      # 54 tile rows: last patch row has 6
    (153600, 13824, 5120, 20, 320),
    (700, 512, 300, 3, 128), (5000, 1024, 1300, 2, 256), (9000, 64, 2304, 1, 192), (100000, 8192, 768, 2, 320),
    (257, 8, 257, 64, 192), (1, 8, 1, 1, 128), (70000, 2048, 256, 7, 320),
])
def test_block_to_tile_map_covers_every_tile_once(shape):
    """The contraction kernels derive (candidate, tile) from the block id alone; the host replay of
    that map must hit every tile of every candidate exactly once, including the regrouped
    incomplete patch row and a short last token chunk."""
    n_tok, c_in, c_out, n_cand, tokens = shape
    bad, blocks = tlq.selftest_tile_map(n_tok, c_in, c_out, n_cand)
    tiles = _launch_tiles(n_tok, c_out, n_cand, tokens)
    assert bad == 0
    assert blocks >= tiles and blocks % 256 == 0
    if tiles >= 20000:
        # the regrouped patch row (3 x 10 of 32 slots, four patches for 32 tiles) leaves < 3 % dead slots
        assert blocks <= 1.03 * tiles
    assert tlq.selftest_tile_map(0, 8, 8, 1)[0] == -1


# (tokens, channels, outputs, candidates, tokens of the launch's tiles): both sides of the rules that pick the tile
# (512 small tiles; whole rounds of 256 blocks; the room for the loss partials of several candidates), launches of one
# to seven token tiles and both sides of the 1024 tiles up to which a launch is dealt in strips
@pytest.mark.parametrize("shape", [
    (2048, 64, 4096, 1, 128), (2048, 64, 4224, 1, 192), (1800, 4096, 4096, 1, 128), (1200, 5120, 13824, 1, 320),
    (1281, 64, 16384, 1, 192), (256, 512, 512, 20, 128), (1300, 72, 11900, 1, 128), (1300, 72, 12000, 1, 320),
    (8192, 64, 8192, 1, 256), (8192, 64, 8193, 1, 320), (1, 64, 5000, 9, 192), (300, 64, 3000, 7, 192),
    (700, 64, 5120, 20, 256), (1200, 5120, 5120, 20, 256), (1024, 64, 2304, 30, 256), (64, 512, 512, 20, 128)])
def test_self_check_reports_the_launch_of_the_library(shape):
    """*blocks is the grid of the launch that the library makes: in strips one eighth of its tiles per XCD in whole
    rounds of 32 blocks, otherwise whole patches of 32 slots."""
    n_tok, c_in, c_out, n_cand, tokens = shape
    bad, blocks = tlq.selftest_tile_map(n_tok, c_in, c_out, n_cand)
    assert bad == 0
    tiles = _launch_tiles(n_tok, c_out, n_cand, tokens)
    if (tiles if tokens == 128 else tiles * tokens // 256) <= 1024:
        assert blocks == -(-(-(-tiles // 8)) // 32) * 256
    else:
        assert blocks % 256 == 0 and tiles <= blocks < 2 * tiles


def test_no_launch_in_a_forked_child(monkeypatch):
    """A forked child has its parent's GPU tensors but no usable GPU state: torch refuses there, before the library is
    called with a stream."""
    import torch
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_isInBadFork", lambda: True)
    monkeypatch.setattr(torch.cuda, "_is_in_bad_fork", lambda: True)
    with pytest.raises(RuntimeError, match="fork"):
        tlq._stream()


def code_objects(blob):
    """The device code objects of the library: entries of its offload bundles."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        p = at + len(magic)
        (n,) = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(n):
            offset, size, name = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + name]
            p += 24 + name
            if triple.startswith(b"hip") and size:
                yield blob[at + offset:at + offset + size]
        at += len(magic)


LOSS, TOK, STORE, DOT = range(4)


def test_only_reachable_contraction_kernels_are_compiled():
    """The library holds the contraction kernels that some call launches and no others (every one lengthens
    the loading of the library): operand type, LDS stages, epilogue (loss, loss with per-token
    errors, store, quadratic form), symmetric form, k tail, 64-row halves of a wave tile; of the wider and narrower tiles
    operand type, epilogue, symmetric form, k tail and token blocks; of the 128 x 64 ones operand type, epilogue and k tail; of
    the 128 x 128 ones with token errors LDS stages and k tail; of the integer ones LDS stages, epilogue, halves and token blocks."""
    blob = open(tlq.LIB_PATH, "rb").read()

    def found(pattern):
        names = {m for m in re.findall(rb"_ZN3tlq\d+" + pattern + rb"EEEvNS_7GemmDevE", blob)}
        return {tuple(int(v) if v.isdigit() else v.decode() for v in m) for m in names}
    ty = rb"INS_[34](F16|BF16)E"
    have = found(rb"gemm_dma_kernel" + ty + rb"Li(\d)ELi(\d)ELb(\d)ELb(\d)ELi(\d)")
    want = set()
    for tail in (0, 1):
        for t in ("F16", "BF16"):
            want |= {(t, 2, epi, 0, tail, 2) for epi in (LOSS, TOK, STORE)}
            want |= {(t, st, STORE, 0, tail, 1) for st in (2, 4)}
        want |= {("F16", st, LOSS, 0, tail, 1) for st in (2, 4)} | {("F16", 2, DOT, 1, tail, 2)}
    assert have == want, (sorted(have - want), sorted(want - have))
    have = found(rb"gemm_width_kernel" + ty + rb"Li(\d)ELb(\d)ELb(\d)ELi(\d)")
    want = {(t, STORE, 0, tail, jb) for t in ("F16", "BF16") for tail in (0, 1) for jb in (3, 5)}
    want |= {("F16", epi, 0, tail, jb) for tail in (0, 1) for epi, jb in ((LOSS, 3), (LOSS, 5), (TOK, 5))}
    want |= {("F16", DOT, 1, tail, 5) for tail in (0, 1)}
    assert have == want, (sorted(have - want), sorted(want - have))
    have = found(rb"gemm_half_kernel" + ty + rb"Li(\d)ELb(\d)")
    want = {(t, epi, tail) for tail in (0, 1) for t, epi in (("F16", LOSS), ("F16", TOK), ("F16", STORE), ("BF16", STORE))}
    assert have == want, (sorted(have - want), sorted(want - have))
    have = found(rb"gemm_small_tok_kernelILi(\d)ELb(\d)")
    want = {(st, tail) for st in (2, 4) for tail in (0, 1)}
    assert have == want, (sorted(have - want), sorted(want - have))
    have = found(rb"gemm_i8_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)")
    want = {(2, epi, 2, jb) for epi in (LOSS, STORE) for jb in (3, 4, 5)} | {(st, epi, 1, 4) for epi in (LOSS, STORE) for st in (2, 4)}
    assert have == want, (sorted(have - want), sorted(want - have))


def test_contraction_kernels_are_loaded_in_five_parts():
    """A code object is loaded as a whole by the first call that needs one of its kernels: square, wider and narrower, 128 x 64,
    128 x 128 with token errors, and integer tiles are one each, and the other kernels of the library are in none of them."""
    families = [rb"gemm_dma_kernel", rb"gemm_width_kernel", rb"gemm_half_kernel", rb"gemm_small_tok_kernel", rb"gemm_i8_kernel",
                rb"quant_row_kernel", rb"xstat_partial_kernel"]
    objects = list(code_objects(open(tlq.LIB_PATH, "rb").read()))
    where = [[i for i, o in enumerate(objects) if f in o] for f in families]
    assert all(len(w) == 1 for w in where) and len({w[0] for w in where}) == len(families), where
