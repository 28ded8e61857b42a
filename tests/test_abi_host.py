"""Host-side checks of the C ABI that need no GPU: the library loads, exports every
symbol the header declares, and rejects bad arguments before touching the device."""
import ctypes
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ea():
    from paper_2105_04779_amd import el_attn
    return el_attn


def test_library_exports_every_declared_symbol(ea):
    header = open(os.path.join(ROOT, "include", "el_attn.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(el_attn_[a-z_]+)\s*\(", header))
    assert declared, "no declarations found in the header"
    assert declared == set(ea.EXPORTED_SYMBOLS)
    for name in declared:
        assert hasattr(ea.lib, name), f"{name} is declared but not exported"


def test_version_and_strings(ea):
    assert ea.el_attn_version() >= 100
    assert ea.el_attn_max_splits() >= 1
    assert ea.status_string(ea.EL_OK) == "ok"
    for s in range(1, 6):
        assert ea.status_string(s) not in ("ok", "unknown status")
    assert ea.status_string(99) == "unknown status"


def _cfg(ea, **kw):
    base = dict(heads=4, d_model=64, d_k=16, dtype=ea.EL_F32, out_dtype=ea.EL_F32,
                max_batch=2, max_beam=2, max_n=32, flags=0)
    base.update(kw)
    return ea.ElAttnConfig(*[base[k] for k in ("heads", "d_model", "d_k", "dtype", "out_dtype",
                                               "max_batch", "max_beam", "max_n", "flags")])


FAKE = ctypes.c_void_p(0x1000)  # never dereferenced: validation fails first


def test_prepare_rejects_bad_arguments_before_any_device_work(ea):
    I, U = ea.EL_ERR_INVALID_ARG, ea.EL_ERR_UNSUPPORTED
    ok = _cfg(ea)
    st, _ = ea.el_attn_prepare(ok, None, None, FAKE, None, FAKE, None, FAKE, None)
    assert st == I
    st, _ = ea.el_attn_prepare(ok, FAKE, None, FAKE, None, FAKE, None, None, None)
    assert st == I
    for bad in (dict(heads=0), dict(d_model=0), dict(d_k=-1), dict(max_batch=0), dict(max_beam=0), dict(max_n=0)):
        st, _ = ea.el_attn_prepare(_cfg(ea, **bad), FAKE, None, FAKE, None, FAKE, None, FAKE, None)
        assert st == I, bad
    for bad in (dict(d_k=8), dict(dtype=7), dict(out_dtype=9), dict(dtype=ea.EL_F16, out_dtype=ea.EL_BF16),
                dict(d_model=16384, heads=256, d_k=64)):
        st, _ = ea.el_attn_prepare(_cfg(ea, **bad), FAKE, None, FAKE, None, FAKE, None, FAKE, None)
        assert st == U, bad


def test_null_context_is_rejected_everywhere(ea):
    I = ea.EL_ERR_INVALID_ARG
    assert ea.el_attn_workspace_bytes(None) == 0
    assert ea.el_attn_bind_workspace(None, FAKE, 1024) == I
    assert ea.el_attn_decode_step(None, FAKE, 64, None, FAKE, FAKE, 1, 1, 1) == I
    assert ea.el_attn_expand_query(None, FAKE, FAKE, 1, 1) == I
    assert ea.el_attn_set_splits(None, 1) == I
    assert ea.el_attn_set_row_groups(None, 1) == I
    assert ea.el_attn_uses_mfma(None) == 0
    assert ea.el_attn_core_timing_enable(None, 4) == I
    assert ea.el_attn_core_timing_read(None, 4)[0] == I
    assert ea.el_attn_destroy(None) == I
    assert ea.el_attn_decode_segment(None, FAKE, 64, None, FAKE, FAKE, FAKE, 1, 1, 1) == I
    assert ea.el_attn_merge_segments(None, 1, [FAKE], [FAKE], FAKE, 1, 1) == I
    assert 1 <= ea.el_attn_max_segments() <= 16


def test_prepare_without_a_device_reports_hip_error(ea):
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is visible")
    st, ctx = ea.el_attn_prepare(_cfg(ea), FAKE, None, FAKE, None, FAKE, None, FAKE, None)
    assert st == ea.EL_ERR_HIP
    assert not ctx.value


def test_gather_batch_rejects_bad_arguments_before_any_device_work(ea):
    I = ea.EL_ERR_INVALID_ARG
    A, B, X = ctypes.c_void_p(0x10000), ctypes.c_void_p(0x20000), ctypes.c_void_p(0x30000)   # never dereferenced

    def call(dtype=ea.EL_BF16, d_model=1024, src=A, sstride=64 * 1024, lsrc=None, bsrc=4,
             dst=B, dstride=64 * 1024, ldst=None, bdst=3, index=X, n=64):
        return ea.el_attn_gather_batch(dtype, d_model, src, sstride, lsrc, bsrc, dst, dstride, ldst, bdst, index, n)

    assert call(src=None) == I and call(dst=None) == I and call(index=None) == I
    assert call(dtype=5) == I
    for bad in (dict(d_model=0), dict(bsrc=0), dict(bdst=0), dict(n=0), dict(bdst=70000)):
        assert call(**bad) == I, bad
    assert call(sstride=64 * 1024 - 8) == I and call(dstride=100) == I          # shorter than n rows
    assert call(d_model=1020) == I                                              # 2040-byte rows: not a multiple of 16
    assert call(dtype=ea.EL_F32, d_model=6, sstride=6 * 64, dstride=6 * 64) == I
    assert call(src=ctypes.c_void_p(0x10008)) == I                              # misaligned
    assert call(sstride=64 * 1024 + 4) == I                                     # batch stride breaks the 16-byte alignment


def test_step_operands_are_validated_on_the_host(ea):
    """The checks decode_step applies to its operands, through the context-free entry point:
    shapes, strides and, on the MFMA path, 16-byte alignment.  Fake pointers, never dereferenced."""
    I, OK = ea.EL_ERR_INVALID_ARG, ea.EL_OK
    H, Q, O, L = (ctypes.c_void_p(v) for v in (0x100000, 0x200000, 0x300000, 0x400000))
    cfg = _cfg(ea, heads=16, d_model=1024, d_k=64, dtype=ea.EL_BF16, max_batch=8, max_beam=4, max_n=128)

    def call(mfma=1, H=H, stride=128 * 1024, lengths=L, queries=Q, out=O, B=8, beam=4, n=128, cfg=cfg):
        return ea.el_attn_check_step_operands(cfg, mfma, H, stride, lengths, queries, out, B, beam, n)

    assert call() == OK and call(lengths=None) == OK and call(mfma=0) == OK
    for bad in (dict(H=None), dict(queries=None), dict(out=None), dict(B=0), dict(B=9), dict(beam=5), dict(n=0), dict(n=129),
                dict(stride=128 * 1024 - 8)):
        assert call(**bad) == I, bad
    off = lambda p, k: ctypes.c_void_p(p.value + k)
    # MFMA path: 16-byte pieces
    for bad in (dict(H=off(H, 2)), dict(H=off(H, 8)), dict(queries=off(Q, 2)), dict(out=off(O, 4)), dict(out=off(O, 8)),
                dict(stride=128 * 1024 + 4), dict(stride=128 * 1024 + 1), dict(lengths=off(L, 2))):
        assert call(**bad) == I, bad
    assert call(stride=128 * 1024 + 8) == OK                     # 16 bytes more between batch elements
    # generic path: element alignment only
    assert call(mfma=0, H=off(H, 2), queries=off(Q, 2), stride=128 * 1024 + 1) == OK
    assert call(mfma=0, H=off(H, 1)) == I and call(mfma=0, out=off(O, 2)) == I and call(mfma=0, lengths=off(L, 1)) == I
    # a shape without MFMA kernels cannot be asked for their rules
    c640 = _cfg(ea, heads=10, d_model=640, d_k=64, dtype=ea.EL_BF16, max_batch=8, max_beam=4, max_n=128)
    assert call(cfg=c640, stride=128 * 640) == ea.EL_ERR_UNSUPPORTED
    assert call(cfg=c640, mfma=0, stride=128 * 640) == OK
    c768 = _cfg(ea, heads=12, d_model=768, d_k=64, dtype=ea.EL_BF16, max_batch=8, max_beam=4, max_n=128)
    assert call(cfg=c768, stride=128 * 768) == OK                # rows of 1.5 KB have MFMA kernels too
    assert ea.lib.el_attn_check_step_operands(None, 1, H, 1, L, Q, O, 1, 1, 1) == I


def test_plan_preview_on_the_benchmark_shapes(ea):
    """The automatic cut of the work, on a 256-unit device: host arithmetic only."""
    def plan(B, beam, heads, d_m, n):
        st, rg, sp = ea.el_attn_plan_preview(B, beam, heads, d_m, n, 256)
        assert st == ea.EL_OK
        return rg, sp

    def short(B, beam, heads, d_m, n):
        return ea.el_attn_plan_short_core(B, B, beam, heads, d_m, n, 256)
    # rows per row block in 16s, spans of the tile list
    assert plan(64, 4, 16, 1024, 1024) == (2, 128)   # 64 rows: two blocks of 32, one workgroup per compute unit
    assert plan(320, 4, 16, 1024, 1024) == (2, 128)  # more sentences: longer spans, never more workgroups than units
    assert plan(512, 1, 16, 1024, 1024) == (1, 256)  # per-beam histories: 16 rows, one block
    assert plan(64, 4, 16, 1024, 256) == (2, 128)    # 1024 tiles: still eight per span
    assert plan(200, 4, 16, 1024, 64) == (2, 128)    # four tiles per sentence, too many for the core of short spans
    # small steps: the core of short spans, four tiles and 16 rows a workgroup
    assert plan(64, 4, 16, 1024, 64) == (1, 64)      # one span per sentence, 4 x 64 workgroups
    assert plan(64, 4, 16, 1024, 32) == (1, 64)
    assert plan(2, 4, 16, 1024, 16) == (1, 2)        # two tiles in all
    assert plan(1, 4, 16, 1024, 613) == (1, 10) and plan(1, 5, 8, 512, 613) == (1, 10)       # 4 x 10 and 3 x 10 workgroups
    assert plan(4, 4, 16, 1024, 410) == (1, 28)
    for B in (1, 3, 17, 64, 100, 1000):
        for beam in (1, 2, 4, 5, 8):
            for n in (1, 16, 100, 1024, 4096):
                rg, sp = plan(B, beam, 16, 1024, n)
                blocks = -(-16 * beam // (16 * rg))
                if short(B, beam, 16, 1024, n):
                    assert rg == 1 and sp == B * -(-n // 64) and sp * blocks <= 2 * 256
                    assert sp <= B * ea.el_attn_max_splits()                   # a span is a piece, and every piece has a slot
                else:
                    assert rg == (1 if beam == 1 else 2) and 1 <= sp and sp * blocks <= max(256, blocks)
                    assert sp <= B * (ea.el_attn_max_splits() - 1)
    # short spans of the streaming core: a block of 32 rows is two workgroups of 16, and still never more workgroups than units
    assert plan(16, 4, 16, 1024, 300) == (2, 64) and plan(12, 4, 16, 1024, 512) == (2, 64)   # 4 x 64 workgroups
    for B in (1, 2, 5, 24, 48):
        for heads, beam, d_m in ((16, 4, 1024), (12, 5, 768), (8, 5, 512), (8, 3, 512), (12, 3, 768)):
            for n in (16, 100, 512, 1024):
                rows, (rg, sp) = heads * beam, plan(B, beam, heads, d_m, n)
                if short(B, beam, heads, d_m, n):
                    continue
                halves = B * -(-n // 16) * -(-rows // 32) <= 6 * 256
                assert rg == 2 and sp * -(-rows // (16 if halves else 32)) <= 256
    I = ea.EL_ERR_INVALID_ARG
    assert ea.el_attn_plan_preview(0, 4, 16, 1024, 64, 256)[0] == I
    assert ea.el_attn_plan_preview(4, 4, 16, 1024, 64, 0)[0] == I
    assert ea.el_attn_plan_preview(4, 4, 10, 640, 64, 256)[0] == ea.EL_ERR_UNSUPPORTED
    assert ea.el_attn_plan_preview(64, 4, 12, 768, 1024, 256)[:2] == (ea.EL_OK, 2)   # 48 rows: two blocks of 32
    assert ea.el_attn_plan_preview(2**31 - 1, 1, 8, 512, 64, 256) == (ea.EL_OK, 1, 2**31 - 1)      # not cut: a span each
    for bad in ((4, 0, 4, 16, 1024, 64, 256), (4, 5, 4, 16, 1024, 64, 256), (4, 4, 4, 10, 640, 64, 256), (4, 4, 4, 16, 1024, 64, 0)):
        assert ea.el_attn_plan_short_core(*bad) == 0


def test_lines_of_the_core_of_short_spans(ea):
    """Which core a step runs on, on both sides of every line of the rule, and what the kernels take for granted of the plan."""
    def short(B, beam, heads, d_m, n, max_batch=None, units=256):
        return ea.el_attn_plan_short_core(max_batch or B, B, beam, heads, d_m, n, units)
    # several spans an element: all workgroups at once
    assert short(8, 4, 16, 1024, 512) and not short(9, 4, 16, 1024, 512)             # 256 and 288 workgroups
    assert short(10, 4, 12, 768, 512) and not short(11, 4, 12, 768, 512)             # 240 and 264
    assert short(16, 4, 8, 512, 512) and not short(17, 4, 8, 512, 512)
    assert short(4, 4, 16, 1024, 512, units=128) and not short(5, 4, 16, 1024, 512, units=128)
    # one span an element: two rounds of them, three at d_m 512
    assert short(128, 4, 16, 1024, 64) and not short(129, 4, 16, 1024, 64) and not short(128, 4, 16, 1024, 65)
    assert short(480, 1, 16, 1024, 64) and not short(481, 1, 16, 1024, 64)           # one row block: 15/8 rounds
    assert short(480, 1, 12, 768, 64) and not short(481, 1, 12, 768, 64)
    assert short(170, 4, 12, 768, 64) and not short(171, 4, 12, 768, 64)
    assert short(384, 4, 8, 512, 64) and not short(385, 4, 8, 512, 64)
    assert short(768, 1, 8, 512, 64) and not short(769, 1, 8, 512, 64)
    assert not short(1024, 1, 8, 512, 64) and short(1024, 1, 8, 512, 64, units=512) and not short(1025, 1, 8, 512, 64, units=512)
    # beyond 13 spans an element: at most three quarters of the compute units in spans
    assert short(19, 1, 16, 1024, 832) and not short(18, 1, 16, 1024, 833) and short(13, 1, 16, 1024, 896)
    assert short(12, 1, 16, 1024, 960) and not short(13, 1, 16, 1024, 960)
    # every piece has a slot: fifteen of an element where the batch is the largest prepared for
    assert short(1, 4, 16, 1024, 960) and not short(1, 4, 16, 1024, 961) and short(1, 4, 16, 1024, 961, max_batch=2)
    # long elements in a context for many: not where this core's cut has more than eight pieces beyond the other one's
    for B in (1, 2, 3):
        assert short(B, 1, 16, 1024, 2500, max_batch=64) and not short(B, 1, 16, 1024, 2800, max_batch=64)
        assert not short(B, 1, 8, 512, 5000, max_batch=64) and not short(B, 1, 8, 512, 12000, max_batch=64)
    assert short(1, 1, 16, 1024, 8192, max_batch=64) and not short(1, 1, 16, 1024, 8200, max_batch=64)     # spans of four tiles either way
    for units in (64, 256, 304):
        for d_m, heads in ((512, 8), (768, 12), (1024, 16), (1024, 8), (768, 24)):
            for beam in (1, 3, 4, 8):
                for n in (1, 16, 17, 64, 65, 128, 500, 832, 833, 960, 1024, 3000):
                    for B in (1, 2, 5, 13, 40, 100, 256, 511, 768, 1024, 1025):
                        for max_batch in (B, 2 * B):
                            if not short(B, beam, heads, d_m, n, max_batch, units):
                                continue
                            spans = B * -(-n // 64)
                            assert B <= 1024 and spans <= 1024 and spans <= 15 * max_batch
                            if max_batch == B:
                                assert ea.el_attn_plan_preview(B, beam, heads, d_m, n, units) == (ea.EL_OK, 1, spans)


def test_plan_of_a_step_is_the_one_launched(ea):
    """el_attn_plan_step on both sides of every line of the wide workgroups' rule (256 compute units): which core, how many
    positions and rows a workgroup takes, how many spans.  The two previews go on describing the choice without them."""
    def plan(B, beam, d_m, n, max_batch=None, units=256):
        st, *p = ea.el_attn_plan_step(max_batch or B, B, beam, d_m // 64, d_m, n, units)
        assert st == ea.EL_OK
        return tuple(p)
    # shapes that the previews have on the streaming core
    assert plan(16, 4, 1024, 300) == (64, 2, 80) and plan(12, 4, 1024, 512) == (64, 2, 96) and plan(64, 4, 512, 512) == (128, 2, 256)
    assert not ea.el_attn_plan_short_core(12, 12, 4, 16, 1024, 512, 256) and ea.el_attn_plan_preview(12, 4, 16, 1024, 512, 256) == (ea.EL_OK, 2, 64)
    # ... or with a second round of the small workgroups: not at d_m 512, and at 1024 only where 32-row blocks pad no further
    assert plan(100, 4, 768, 64) == (96, 2, 100) and plan(100, 5, 768, 64) == (96, 2, 100)
    assert plan(128, 4, 1024, 64) == (64, 2, 128) and plan(100, 3, 1024, 64) == (64, 1, 100)
    assert plan(200, 4, 512, 64) == (64, 1, 200)
    # one round of the small workgroups stays theirs, one round of the wide ones is the end
    assert plan(16, 4, 512, 512) == (64, 1, 128) and plan(17, 4, 512, 512) == (128, 2, 68)
    assert plan(65, 4, 512, 512)[0] == 0 and plan(64, 1, 512, 512) == (128, 1, 256) and plan(65, 1, 512, 512)[0] == 0
    assert plan(85, 1, 768, 288) == (96, 1, 255) and plan(86, 1, 768, 288)[0] == 0
    assert plan(32, 4, 1024, 256) == (64, 2, 128) and plan(33, 4, 1024, 256)[0] == 0
    assert plan(64, 4, 512, 512, units=304) == (128, 2, 256) and plan(76, 4, 512, 512, units=304) == (128, 2, 304) and plan(77, 4, 512, 512, units=304)[0] == 0
    # one row block and many spans of an element
    assert plan(38, 2, 1024, 320) == (64, 2, 190) and plan(39, 2, 1024, 320)[0] == 0 and plan(64, 2, 1024, 256) == (64, 2, 256)
    assert plan(25, 1, 768, 960) == (96, 1, 250) and plan(23, 1, 768, 961)[0] == 0
    assert plan(19, 2, 768, 1248) == (96, 2, 247) and plan(18, 2, 768, 1249)[0] == 0
    assert plan(512, 1, 1024, 1024) == (0, 1, 256) and plan(64, 4, 1024, 1024) == (0, 2, 128)
    # d_m 1024 and 16 rows: nothing wider
    assert plan(300, 1, 1024, 64) == (64, 1, 300) and plan(260, 1, 1024, 65)[0] == 0
    tiles = {512: 128, 768: 96, 1024: 64}
    for units in (64, 256, 304):
        for d_m in (512, 768, 1024):
            for beam in (1, 2, 3, 4, 5, 8):
                for n in (1, 16, 64, 65, 96, 97, 128, 129, 300, 512, 960, 1024, 3000):
                    for B in (1, 5, 13, 32, 64, 100, 200, 256, 300, 1024, 1025):
                        for max_batch in (B, 2 * B):
                            positions, groups, spans = plan(B, beam, d_m, n, max_batch, units)
                            rows = beam * d_m // 64
                            small = ea.el_attn_plan_short_core(max_batch, B, beam, d_m // 64, d_m, n, units)
                            if positions == 0:
                                assert not small and groups in (1, 2) and spans >= 1
                            elif small and (positions, groups) == (64, 1):
                                assert spans == B * -(-n // 64) <= min(1024, 15 * max_batch)
                            else:
                                assert positions == tiles[d_m] and groups == (2 if rows > 16 else 1) and (positions, groups) != (64, 1)
                                assert spans == B * -(-n // positions) and spans * -(-rows // (16 * groups)) <= units and spans <= 13 * B
    I = ea.EL_ERR_INVALID_ARG
    assert ea.el_attn_plan_step(4, 5, 4, 16, 1024, 64, 256)[0] == I and ea.el_attn_plan_step(4, 4, 4, 16, 1024, 64, 0)[0] == I
    assert ea.el_attn_plan_step(4, 4, 4, 10, 640, 64, 256)[0] == ea.EL_ERR_UNSUPPORTED
    assert ea.lib.el_attn_plan_step(4, 4, 4, 16, 1024, 64, 256, None, ctypes.byref(ctypes.c_int32()), ctypes.byref(ctypes.c_int32())) == I


def test_single_queries_of_one_length_stay_on_the_streaming_core(ea):
    """d_m 512, one query per history, a span each on more than 15/16 of the compute units: an element a workgroup on either core, and
    the streaming core is the faster one."""
    def positions(B, beam, n, d_m=512, units=256):
        return ea.el_attn_plan_step(B, B, beam, d_m // 64, d_m, n, units)[1]
    assert positions(240, 1, 128) == 128 and positions(241, 1, 128) == 0 and positions(256, 1, 128) == 0 and positions(257, 1, 128) == 0
    assert positions(241, 1, 65) == 0 and positions(241, 1, 64) == 64 and positions(128, 1, 129) == 128 and positions(285, 1, 128, units=304) == 128
    assert positions(256, 2, 128) == positions(256, 3, 128) == positions(256, 4, 128) == 128
    assert positions(256, 1, 96, d_m=768) == 96


def test_check_inputs_rejects_bad_arguments_before_any_device_work(ea):
    I = ea.EL_ERR_INVALID_ARG
    A, Rp = ctypes.c_void_p(0x10000), ctypes.c_void_p(0x20000)   # never dereferenced

    def call(dtype=ea.EL_BF16, d_model=1024, H=A, stride=64 * 1024, lengths=None, B=4, n=64, report=Rp):
        return ea.el_attn_check_inputs(dtype, d_model, H, stride, lengths, B, n, report)

    assert call(H=None) == I and call(report=None) == I
    assert call(dtype=9) == I
    for bad in (dict(d_model=0), dict(B=0), dict(n=0), dict(B=70000)):
        assert call(**bad) == I, bad
    assert call(stride=64 * 1024 - 8) == I                      # shorter than n rows
    assert call(d_model=1020) == I                              # rows not a multiple of 16 bytes
    assert call(H=ctypes.c_void_p(0x10008)) == I                # misaligned H
    assert call(report=ctypes.c_void_p(0x20004)) == I           # misaligned report


def test_build_fails_on_register_spills_in_the_attention_core():
    """The build reads hipcc's resource remarks back: spills in any instance of the core kernel are reported,
    spills elsewhere and clean instances are not."""
    from paper_2105_04779_amd import build
    core = "_ZN2el13k_core_streamILi1024ELb1ELi2ELb0EEEvNS_10StreamArgsE"
    remarks = "\n".join([
        f"core_stream.hip:95:1: remark: Function Name: {core} [-Rpass-analysis=kernel-resource-usage]",
        "core_stream.hip:95:1: remark:     VGPRs: 256 [-Rpass-analysis=kernel-resource-usage]",
        "core_stream.hip:95:1: remark:     VGPRs Spill: 5 [-Rpass-analysis=kernel-resource-usage]",
        "core_stream.hip:95:1: remark: Function Name: _ZN2el13k_core_streamILi512ELb0ELi1ELb0EEEvNS_10StreamArgsE [-R]",
        "core_stream.hip:95:1: remark:     VGPRs Spill: 0 [-R]",
        "gemm_mfma.hip:70:1: remark: Function Name: _ZN2el11k_gemm_slabILb1ELi1EEEvNS_8GemmArgsE [-R]",
        "gemm_mfma.hip:70:1: remark:     VGPRs Spill: 9 [-R]",
    ])
    assert build.check_core_spills(remarks) == {core: 5}
    assert build.check_core_spills("") == {}


@pytest.mark.parametrize("kernel", ["k_qelqILi1024ELb1ELi4EE", "k_vprojILi1024ELi4ELb1EE", "k_oprojILi768ELi2EfE", "k_small_stepIffLi128EE"])
def test_build_fails_on_register_spills_where_weights_live_in_registers(kernel):
    from paper_2105_04779_amd import build
    name = "_ZN2el%d%sEvNS_1AE" % (len(kernel), kernel)
    block = "a.hip:1:1: remark: Function Name: %s [-R]\na.hip:1:1: remark:     SGPRs Spill: 3 [-R]\na.hip:1:1: remark:     VGPRs Spill: %d [-R]\n"
    assert build.check_core_spills(block % (name, 2)) == {name: 2}
    assert build.check_core_spills(block % (name, 0)) == {}


def test_the_query_kernel_waits_for_nothing_before_all_of_it_is_requested(tmp_path):
    """In every instance of k_qelq the lengths, the bias, the rows and both weight slices are under way before the first wait for
    memory: looked at earlier, each is a round trip of its own in front of the cut and of the first product."""
    from paper_2105_04779_amd import build
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    asm = tmp_path / "gemm_mfma.s"
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *flags, "-S", "--cuda-device-only", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    "-o", str(asm), os.path.join(build.CSRC, "gemm_mfma.hip")], check=True, capture_output=True)
    bodies = re.findall(r"^_ZN2el6k_qelqILi(\d+)ELb\dELi(\d)E\S*:\s(.*?)\.end_amdhsa_kernel", asm.read_text(), re.S | re.M)
    assert len(bodies) == 14
    for d_m, parts, body in bodies:
        slices = int(d_m) // 256
        loads = 2 + 1 + slices + 4 * slices + 4 * int(parts)         # lengths, bias, rows, W^Q, W^K
        before = body[:re.search(r"s_waitcnt[^\n]*vmcnt", body).start()]
        assert before.count("global_load") == loads, (d_m, parts, before.count("global_load"))


def test_short_core_counts_its_requests(tmp_path):
    """k_core_short waits for its tiles by count: as many vector loads as EL-Q fragments are requested behind the last tile, nothing
    else, and the first read of LDS follows that wait."""
    from paper_2105_04779_amd import build
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    asm = tmp_path / "core_short.s"
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *flags, "-S", "--cuda-device-only", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    "-o", str(asm), os.path.join(build.CSRC, "core_short.hip")], check=True, capture_output=True)
    bodies = re.findall(r"^_ZN2el12k_core_shortILi(\d+)ELb\dELi\dELi(\d)E\S*:\s(.*?)\.end_amdhsa_kernel", asm.read_text(), re.S | re.M)
    assert len(bodies) == 16
    for d_m, blocks, body in bodies:
        loads = 2 * (int(d_m) // 256) * int(blocks)                  # both planes of each 32-column chunk of a wavefront, per 16 rows
        # the wait is written out (the compiler's own have no marks around them); the block that it ends starts behind the last tile
        wait = re.search(r"ASMSTART\s+s_waitcnt vmcnt\((\d+)\)", body)
        assert int(wait.group(1)) == loads, (d_m, blocks, wait.group(0))
        block = re.split(r"^\.LBB\S+:", body[:wait.start()], flags=re.M)[-1].rsplit("global_load_lds_dwordx4", 1)[-1]
        assert len(re.findall(r"^\s*(?:global|buffer|flat|scratch)_(?:load|store)", block, re.M)) == loads, (d_m, blocks)
        assert "ds_read" not in body[:wait.start()]


def test_fp32_products_leave_room_for_workgroups(tmp_path):
    """k_gemm_f32 in the forms for more workgroups than run at once: registers for four workgroups of eight wavefronts on a compute
    unit (16 x 16 outputs), three (32 x 16) or two (32 x 32), whatever the types and the alignment; 512 registers a lane of a SIMD
    and two of a workgroup's wavefronts on each.  Rows held across the wait for the length cost one of them."""
    from paper_2105_04779_amd import build
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    res = subprocess.run([hipcc, *flags, "-S", "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-I", os.path.join(build.ROOT, "include"),
                          "-I", build.CSRC, "-o", str(tmp_path / "generic.s"), os.path.join(build.CSRC, "generic_kernels.hip")],
                         check=True, capture_output=True, text=True)
    found = re.findall(r"Function Name: (\S*k_gemm_f32I\S*?Lb\dELi(\d)ELi(\d)E\S*).*?VGPRs: (\d+)", res.stderr, re.S)
    forms = set()
    for name, rows, cols, registers in found:
        form = re.search(r"GemmFormE(\d)", name)
        forms.add((rows, cols, form and form.group(1)))
        if form and form.group(1) == "0":                            # early: all workgroups run at once
            continue
        assert int(registers) <= {("1", "1"): 64, ("2", "1"): 80, ("2", "2"): 128}[rows, cols], (name, registers)
    assert forms == {("1", "1", "0"), ("1", "1", "2"), ("2", "1", "0"), ("2", "1", "1"), ("2", "1", "2"), ("2", "2", "1"), ("2", "2", "2")}
