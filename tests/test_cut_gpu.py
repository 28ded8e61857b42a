"""GPU parity of the decode step where the cut of its work changes form: one element cut into many spans, few elements
cut one by one, spans that run through more elements than the table lists lengths for, and dozens of pieces per element;
with the projections' column splits and row-tile groups that belong to these row counts."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_2105_04779_amd import el_attn, workloads as wl
from helpers import TOL, gpu_out, make_layer, oracle_out, record, rel_err, to_device

pytestmark = pytest.mark.gpu


def compute_units():
    return torch.cuda.get_device_properties(0).multi_processor_count

CASES = [
    # dtype, B, beam, heads, d_m, n, lens, splits; where a step with splits 0 runs on the core of short spans, it is run on the
    # streaming core (whose own per-element cut these were written for) as well
    ("bf16", 1, 4, 16, 1024, 1000, [1000], 0),              # one sentence: 13 spans of five tiles, as many pieces to merge
    ("bf16", 1, 4, 16, 1024, 613, [613], 0),
    ("f16", 1, 1, 8, 512, 333, [333], 0),
    ("bf16", 1, 3, 12, 768, 17, [17], 0),                   # two tiles, the second with one row
    ("bf16", 4, 4, 16, 1024, 410, [410, 205, 1, 333], 0),   # cut per element
    ("f16", 5, 5, 12, 768, 300, [300, 16, 17, 299, 1], 0),
    ("bf16", 2, 4, 16, 1024, 700, [700, 350], 15),          # the most splits
    ("bf16", 2, 2, 8, 512, 500, [1, 500], 15),
    ("bf16", 700, 4, 16, 1024, 40, "mixed", 0),             # more than four elements per span, some of one row
    ("f16", 1000, 2, 8, 512, 33, "mixed", 0),
    ("bf16", 33, 5, 12, 768, 90, "mixed", 0),               # 165 rows: a last row tile of five
    ("bf16", 24, 4, 16, 1024, 512, [500] * 23 + [512], 0),  # the longest spans of 16-row workgroups, and one tile beyond them
    ("bf16", 24, 4, 16, 1024, 528, [500] * 23 + [528], 0),
    ("f16", 6, 5, 8, 512, 150, "mixed", 0),                 # 40 rows: three blocks of 16
    ("bf16", 320, 4, 16, 1024, 24, "mixed", 0),             # several row tiles per workgroup of the projections
]


@pytest.mark.parametrize("dtype,B,beam,heads,d_m,n,lens,splits", CASES)
def test_cuts(dtype, B, beam, heads, d_m, n, lens, splits):
    w = wl.custom(f"cut_{dtype}_{B}x{beam}_{d_m}_{n}", dtype=dtype, B=B, beam=beam, heads=heads, d_m=d_m, d_k=64, n=n, index=95)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    L = np.asarray([1 + (b * 13) % n for b in range(B)] if isinstance(lens, str) else lens, dtype=np.int32)
    L[0] = n if isinstance(lens, str) else L[0]
    ref = oracle_out(w, W, H, Q, L)
    for b in range(B):
        H[b, L[b]:] = np.nan
    layer = make_layer(w, W)
    assert layer.uses_mfma
    if splits:
        layer.set_splits(splits)
    short = not splits and el_attn.el_attn_plan_short_core(B, B, beam, heads, d_m, n, compute_units())
    for groups in (0, 1, 2) if short else (0,):
        layer.set_row_groups(groups)
        err = rel_err(gpu_out(layer, w, H, Q, L), ref)
        record(f"{w.name}: splits={splits} row groups={groups} short={short and not groups} err={err:.3e}")
        assert err <= TOL[dtype]
    layer.close()


@pytest.mark.parametrize("heads,d_m", [(16, 1024), (12, 768)])
def test_a_piece_of_vanishing_weight_is_not_multiplied(heads, d_m):
    """Every head scores its last key +512 and the others -512, whose weights underflow to zero in fp32.  The other keys hold
    finite bf16 values beyond the fp16 range, so a piece without the last key stores infinities; its weight is exactly
    zero, and so must its contribution be."""
    w = wl.custom(f"cut_zero_weight_{d_m}", dtype="bf16", B=1, beam=1, heads=heads, d_m=d_m, d_k=64, n=256, index=96)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    L = np.asarray([w.n], dtype=np.int32)
    # projected queries of ones against W^K's first row of ones: a score is 64 / sqrt(64) times the key's first element
    W["Wq"][:] = 0.0
    W["bq"][:] = 1.0
    W["Wk"][:] = 0.0
    W["Wk"][0, :] = 1.0
    H[0, :, 0] = -64.0
    H[0, -1, 0] = 64.0
    H[0, :-1, 1:] = 131072.0
    ref = oracle_out(w, W, H, Q, L)
    layer = make_layer(w, W)
    layer.set_splits(8)
    err = rel_err(gpu_out(layer, w, H, Q, L), ref)
    record(f"{w.name}: err={err:.3e}")
    assert err <= TOL["bf16"]
    layer.close()


@pytest.mark.parametrize("dtype,heads,d_m,beam,n", [("bf16", 16, 1024, 4, 128), ("f16", 8, 512, 1, 128), ("f16", 12, 768, 2, 128)])
def test_cutting_an_element_costs_no_precision(dtype, heads, d_m, beam, n):
    """The same elements as one piece each and as two pieces of four tiles, both on the streaming core.  A piece is rounded to
    fp16 either way; if merged sums were rounded to fp16 once more, the error of X would be sqrt(2) times that of one piece
    and the result's about 1.1 times (measured: 1.08 to 1.13).  Over at least 8000 results the estimate of the ratio scatters
    by 1 % to 2 %.  The core of short spans, which the automatic choice takes for them, has the same two pieces and the same
    roundings (high + low operands, fp32 sums, fp16 pieces), so the same bound holds for it."""
    w = wl.custom(f"cut_precision_{dtype}_{d_m}", dtype=dtype, B=1, beam=beam, heads=heads, d_m=d_m, d_k=64, n=n, index=97)
    W = wl.weights(w)
    L = np.asarray([n], dtype=np.int32)
    assert el_attn.el_attn_plan_short_core(1, 1, beam, heads, d_m, n, compute_units())
    layer = make_layer(w, W)
    err = {0: 0.0, 1: 0.0, 2: 0.0}                     # automatic: the core of short spans
    for k in range(16):
        H, Q, _ = wl.batch(replace(w, index=400 + k), poison=False)
        ref = oracle_out(w, W, H, Q, L)
        for splits in err:
            layer.set_splits(splits)
            d = gpu_out(layer, w, H, Q, L).astype(np.float64) - ref
            err[splits] += float((d * d).sum())
    two, short = (err[2] / err[1]) ** 0.5, (err[0] / err[1]) ** 0.5
    record(f"{w.name}: rms error of two pieces / of one = {two:.4f}, of the core of short spans {short:.4f}")
    assert two <= 1.04 and short <= 1.04
    layer.close()


@pytest.mark.parametrize("dtype,heads,d_m,beam,n", [("f16", 8, 512, 4, 4096), ("bf16", 12, 768, 1, 4093)])
def test_dozens_of_pieces_of_one_element(dtype, heads, d_m, beam, n):
    """A workspace for 64 elements and a call with one: 64 spans of four tiles, all of the same element, merged four pieces at a
    time; the step and the segment form, on the core of short spans, which the automatic choice takes, and on the streaming core."""
    w = wl.custom(f"cut_pieces_{dtype}_{d_m}", dtype=dtype, B=1, beam=beam, heads=heads, d_m=d_m, d_k=64, n=n, index=98)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    L = np.asarray([n], dtype=np.int32)
    st, _, spans = el_attn.el_attn_plan_preview(1, beam, heads, d_m, n, 256)
    assert st == el_attn.EL_OK and spans <= 14                       # with room for one element only
    assert el_attn.el_attn_plan_short_core(64, 1, beam, heads, d_m, n, compute_units())
    ref = oracle_out(w, W, H, Q, L)
    ref_A, ref_lse = oracle.segment_reference(H, L, Q, W["Wq"], W["bq"], W["Wk"], W["bk"], W["Wv"], W["bv"], heads=heads, d_k=64)
    layer = make_layer(w, W, max_batch=64)
    for groups in (0, 1):
        layer.set_row_groups(groups)
        err = rel_err(gpu_out(layer, w, H, Q, L), ref)
        A, lse = layer.decode_segment(to_device(H, dtype), torch.from_numpy(L).cuda(), to_device(Q, dtype))
        torch.cuda.synchronize()
        err_A, err_lse = rel_err(A.cpu().numpy(), ref_A), float(np.abs(lse.cpu().numpy() - ref_lse).max())
        record(f"{w.name}: row groups={groups} err={err:.3e} seg_A err={err_A:.3e} lse err={err_lse:.3e}")
        assert err <= TOL[dtype] and err_A <= TOL[dtype] and err_lse <= 5e-3
    layer.close()


@pytest.mark.parametrize("dtype,d_m,B,beam,n,max_batch", [
    ("bf16", 1024, 1, 1, 960, 1),          # one row, fifteen pieces side by side
    ("f16", 512, 1, 2, 4096, 64),          # two rows, 64 pieces: four rounds of sixteen
    ("bf16", 512, 1, 7, 11000, 96),        # seven rows and more rounds than are in flight
    ("bf16", 1024, 4, 4, 410, 4),          # an element of four rows a tile
    ("f16", 768, 3, 5, 500, 3),            # tiles of four that straddle elements, the last one of three rows
    ("f16", 1024, 2, 4, 500, 2),           # tiles of two rows, eight pieces
    ("bf16", 768, 7, 3, 300, 7),           # 21 rows in tiles of eight
    ("f16", 1024, 9, 5, 640, 9),           # 45 rows in tiles of eight, two column parts
    ("bf16", 512, 16, 8, 130, 16),         # 128 rows in tiles of 16
])
def test_rows_and_pieces_side_by_side(dtype, d_m, B, beam, n, max_batch):
    """Few query rows: the merge takes fewer than 16 of them a workgroup and several pieces of each at a time; elements of one
    piece next to elements of many, lengths from 1 up, step and segment form against the oracle at the step's bar."""
    heads = d_m // 64
    w = wl.custom(f"rows_pieces_{dtype}_{d_m}_{B}x{beam}_{n}", dtype=dtype, B=B, beam=beam, heads=heads, d_m=d_m, d_k=64, n=n, index=101)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    L = np.asarray([n if b == B - 1 else 1 + (b * 77) % n for b in range(B)], dtype=np.int32)
    ref = oracle_out(w, W, H, Q, L)
    ref_A, ref_lse = oracle.segment_reference(H, L, Q, W["Wq"], W["bq"], W["Wk"], W["bk"], W["Wv"], W["bv"], heads=heads, d_k=64)
    for b in range(B):
        H[b, L[b]:] = np.nan
    layer = make_layer(w, W, max_batch=max_batch)
    for splits in (0, 15):
        layer.set_splits(splits)
        err = rel_err(gpu_out(layer, w, H, Q, L), ref)
        A, lse = layer.decode_segment(to_device(H, dtype), torch.from_numpy(L).cuda(), to_device(Q, dtype))
        torch.cuda.synchronize()
        err_A, err_lse = rel_err(A.cpu().numpy(), ref_A), float(np.abs(lse.cpu().numpy() - ref_lse).max())
        record(f"{w.name}: splits={splits} err={err:.3e} seg_A err={err_A:.3e} lse err={err_lse:.3e}")
        assert err <= TOL[dtype] and err_A <= TOL[dtype] and err_lse <= 5e-3
    layer.close()


@pytest.mark.parametrize("dtype,d_m,B,beam,n", [("bf16", 1024, 130, 2, 480), ("f16", 768, 120, 3, 480), ("bf16", 512, 270, 2, 640)])
def test_row_tiles_of_one_and_of_many_rounds(dtype, d_m, B, beam, n):
    """More query rows than the merge has workgroups for in tiles of 16 (256, 336 and 512), one element of as many as thirty pieces
    among elements of a single one, at the start, in the middle and at the end: a workgroup folds in more rounds of a tile than it
    has in flight, before and after tiles of one round.  Step and segment form against the oracle at the step's bar."""
    heads = d_m // 64
    assert B * beam > 16 * (compute_units() // heads)
    w = wl.custom(f"row_tiles_{dtype}_{d_m}", dtype=dtype, B=B, beam=beam, heads=heads, d_m=d_m, d_k=64, n=n, index=105)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    Hd, Qd = to_device(H, dtype), to_device(Q, dtype)
    layer = make_layer(w, W)
    for at in (0, B // 2, B - 1):
        L = np.asarray([n if b == at else 1 + (b * 7) % 16 for b in range(B)], dtype=np.int32)
        Ld = torch.from_numpy(L).cuda()
        ref = oracle_out(w, W, H, Q, L)
        ref_A, ref_lse = oracle.segment_reference(H, L, Q, W["Wq"], W["bq"], W["Wk"], W["bk"], W["Wv"], W["bv"], heads=heads, d_k=64)
        err = rel_err(layer.decode_step(Hd, Ld, Qd).float().cpu().numpy(), ref)
        A, lse = layer.decode_segment(Hd, Ld, Qd)
        err_A, err_lse = rel_err(A.cpu().numpy(), ref_A), float(np.abs(lse.cpu().numpy() - ref_lse).max())
        long = rel_err(A.cpu().numpy()[at * beam:(at + 1) * beam], ref_A[at * beam:(at + 1) * beam])
        record(f"{w.name}: long element {at} err={err:.3e} seg_A err={err_A:.3e} (its own {long:.3e}) lse err={err_lse:.3e}")
        # (the long element's head outputs are small beside those of one position: held to the bar by themselves as well)
        assert err <= TOL[dtype] and err_A <= TOL[dtype] and long <= TOL[dtype] and err_lse <= 5e-3
    layer.close()


SHORT = [
    # dtype, B, beam, heads, d_m, n, lens: at most 256 workgroups of 64 positions and 16 rows (two or three times as many where n <= 64)
    ("bf16", 5, 4, 16, 1024, 200, [200, 1, 16, 17, 64]),            # spans of one to four tiles, of one position and of a full tile
    ("f16", 6, 3, 16, 1024, 129, [129, 128, 127, 113, 65, 48]),     # 48 rows; a span of one position behind full ones
    ("bf16", 9, 5, 12, 768, 130, [130, 80, 81, 33, 32, 31, 97, 2, 64]),   # 60 rows: a block of twelve; the 32-column window
    ("f16", 4, 1, 12, 768, 63, [63, 49, 15, 1]),                    # 12 rows, one span each
    ("f16", 7, 3, 8, 512, 250, [250, 249, 193, 192, 66, 5, 160]),   # 24 rows
    ("bf16", 3, 1, 8, 512, 64, None),                               # 8 rows, no lengths
    ("bf16", 64, 4, 16, 1024, 64, "mixed"),                         # 256 workgroups of one span
    ("bf16", 1, 4, 16, 1024, 960, [947]),                           # fifteen pieces of one element: as many as there are slots
    ("bf16", 400, 1, 16, 1024, 64, "mixed"),                        # a second round of workgroups
    ("f16", 130, 4, 12, 768, 50, "mixed"),
    ("f16", 700, 1, 8, 512, 64, "mixed"),                           # a third, and elements beyond the 512th in the cut
]


@pytest.mark.parametrize("dtype,B,beam,heads,d_m,n,lens", SHORT)
def test_short_spans(dtype, B, beam, heads, d_m, n, lens):
    """The core of short spans against the oracle and against the streaming core (which a set row-group count leaves in charge) on
    the same call: a batch stride beyond n rows, poisoned rows past the lengths, step and segment form.  Both round the pieces to
    fp16 once, elsewhere: they agree to twice the bar of either."""
    w = wl.custom(f"short_{dtype}_{B}x{beam}_{d_m}_{n}", dtype=dtype, B=B, beam=beam, heads=heads, d_m=d_m, d_k=64, n=n, index=99)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    L = np.full(B, n, dtype=np.int32) if lens is None else np.asarray([1 + (b * 13) % n for b in range(B)] if isinstance(lens, str) else lens, dtype=np.int32)
    ref = oracle_out(w, W, H, Q, L)
    wide = np.full((B, n + 3, d_m), np.nan, dtype=np.float32)
    for b in range(B):
        wide[b, :L[b]] = H[b, :L[b]]
    Hd, Qd = to_device(wide, dtype)[:, :n], to_device(Q, dtype)
    Ld = None if lens is None else torch.from_numpy(L).cuda()
    assert el_attn.el_attn_plan_short_core(B, B, beam, heads, d_m, n, compute_units())
    outs = []
    for groups in (0, 1):
        layer = make_layer(w, W)
        layer.set_row_groups(groups)
        y = layer.decode_step(Hd, Ld, Qd).float().cpu().numpy()
        A, lse = layer.decode_segment(Hd, Ld, Qd)
        outs.append((y, A.cpu().numpy(), lse.cpu().numpy()))
        layer.close()
    err = rel_err(outs[0][0], ref)
    record(f"{w.name}: err={err:.3e} streaming core {rel_err(outs[1][0], ref):.3e}")
    assert err <= TOL[dtype]
    for a, b in zip(*outs):
        assert rel_err(a, b) <= 2 * TOL[dtype]


WIDE = [
    # dtype, B, beam, heads, d_m, n, lens: more than 256 workgroups of 64 positions and 16 rows, at most 256 of 128 (d_m 512) or 96
    # (d_m 768) positions and, beyond 16 rows, of 32
    ("f16", 100, 1, 8, 512, 256, "mixed"),                          # 8 rows, spans of one to eight tiles
    ("bf16", 70, 4, 8, 512, 250, "mixed"),                          # 32 rows
    ("f16", 60, 3, 8, 512, 300, "mixed"),                           # 24 rows: half a row group of padding
    ("bf16", 50, 5, 8, 512, 129, [129, 128, 113, 64, 65, 1, 80, 16, 17, 97] * 5),   # 40 rows: two blocks; spans of one position
    ("bf16", 100, 1, 12, 768, 190, "mixed"),                        # 12 rows, spans of one to six tiles
    ("f16", 60, 2, 12, 768, 290, "mixed"),                          # 24 rows
    ("bf16", 30, 5, 12, 768, 300, [300, 97, 96, 95, 64, 65, 1, 33, 193, 16] * 3),   # 60 rows: two blocks, the second of 28
    ("f16", 120, 3, 12, 768, 96, None),                             # 36 rows, one span each, no lengths
    ("bf16", 100, 5, 12, 768, 64, "mixed"),                         # instead of a second round of the small workgroups
    ("bf16", 31, 4, 16, 1024, 250, "mixed"),                        # 64 rows: two blocks of 32, four tiles
    ("f16", 70, 2, 16, 1024, 129, "mixed"),                         # 32 rows
    ("bf16", 24, 5, 16, 1024, 150, [150, 1, 64, 65, 80, 129] * 4),  # 80 rows: the last block half empty
]


@pytest.mark.parametrize("dtype,B,beam,heads,d_m,n,lens", WIDE)
def test_wide_short_spans(dtype, B, beam, heads, d_m, n, lens):
    """The wide workgroups of the core of short spans against the oracle and against the streaming core on the same call, twice
    with the same bits."""
    positions, rows = {512: 128, 768: 96, 1024: 64}[d_m], heads * beam
    block = 32 if rows > 16 else 16
    units = compute_units()
    assert B * -(-n // 64) * -(-rows // 16) > units >= B * -(-n // positions) * -(-rows // block)
    w = wl.custom(f"wide_{dtype}_{B}x{beam}_{d_m}_{n}", dtype=dtype, B=B, beam=beam, heads=heads, d_m=d_m, d_k=64, n=n, index=103)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    L = np.full(B, n, dtype=np.int32) if lens is None else np.asarray([1 + (b * 13) % n for b in range(B)] if isinstance(lens, str) else lens, dtype=np.int32)
    ref = oracle_out(w, W, H, Q, L)
    far = np.full((B, n + 3, d_m), np.nan, dtype=np.float32)
    for b in range(B):
        far[b, :L[b]] = H[b, :L[b]]
    Hd, Qd = to_device(far, dtype)[:, :n], to_device(Q, dtype)
    Ld = None if lens is None else torch.from_numpy(L).cuda()
    outs = []
    for groups in (0, 1):
        layer = make_layer(w, W)
        layer.set_row_groups(groups)
        y = layer.decode_step(Hd, Ld, Qd)
        assert torch.equal(y, layer.decode_step(Hd, Ld, Qd))
        A, lse = layer.decode_segment(Hd, Ld, Qd)
        outs.append((y.float().cpu().numpy(), A.cpu().numpy(), lse.cpu().numpy()))
        layer.close()
    err = rel_err(outs[0][0], ref)
    record(f"{w.name}: err={err:.3e} streaming core {rel_err(outs[1][0], ref):.3e}")
    assert err <= TOL[dtype]
    for a, b in zip(*outs):
        assert rel_err(a, b) <= 2 * TOL[dtype]


@pytest.mark.parametrize("dtype,B,beam,heads,d_m,n,lens", WIDE)
def test_wide_cases_run_on_wide_workgroups(dtype, B, beam, heads, d_m, n, lens):
    """The cases above are launched on the wide workgroups of this device, and not on a core that would pass them as well."""
    positions, rows = {512: 128, 768: 96, 1024: 64}[d_m], heads * beam
    assert el_attn.el_attn_plan_step(B, B, beam, heads, d_m, n, compute_units()) == (el_attn.EL_OK, positions, 2 if rows > 16 else 1, B * -(-n // positions))


@pytest.mark.parametrize("dtype,B,beam,heads,d_m,n", [("bf16", 33, 5, 12, 768, 90), ("f16", 16, 4, 16, 1024, 300)])
def test_streaming_core_of_shapes_of_the_wide_workgroups(dtype, B, beam, heads, d_m, n):
    """Shapes whose automatic choice is the wide workgroups, on the streaming core with row blocks of 16 and of 32."""
    assert el_attn.el_attn_plan_step(B, B, beam, heads, d_m, n, compute_units())[1:3] == ({768: 96, 1024: 64}[d_m], 2)
    w = wl.custom(f"wide_streamed_{dtype}_{B}x{beam}_{d_m}_{n}", dtype=dtype, B=B, beam=beam, heads=heads, d_m=d_m, d_k=64, n=n, index=104)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    L = np.asarray([n if b == 0 else 1 + (b * 13) % n for b in range(B)], dtype=np.int32)
    ref = oracle_out(w, W, H, Q, L)
    for b in range(B):
        H[b, L[b]:] = np.nan
    layer = make_layer(w, W)
    for groups in (0, 1, 2):
        layer.set_row_groups(groups)
        err = rel_err(gpu_out(layer, w, H, Q, L), ref)
        record(f"{w.name}: row groups={groups} err={err:.3e}")
        assert err <= TOL[dtype]
    layer.close()
