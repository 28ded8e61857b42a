"""GPU parity of the fp32-arithmetic path at the sizes where its kernels change form: contraction lengths that are no
multiple of 16 or of 4, operands aligned to one element only, more positions than one chunk of the softmax, keys too
long for scores in memory, the three tile sizes of the products, and the one-launch step at its edges."""
import numpy as np
import pytest

import oracle
from paper_2105_04779_amd import workloads as wl
from helpers import TOL, err_report, fmt_report, gpu_out, make_layer, oracle_out, record, rel_err, to_device

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, B, beam, heads, d_m, d_k, n, lens
    ("f32", 2, 3, 3, 30, 10, 37, [37, 1]),               # nothing divides anything
    ("f32", 3, 2, 5, 100, 20, 61, [61, 16, 17]),         # multiples of 4, not of 16
    ("f32", 2, 4, 5, 320, 64, 1100, [1100, 513]),        # three chunks of 512 positions; a chunk of one position
    ("f32", 2, 16, 4, 64, 16, 600, [600, 599]),          # n > 8 d_m with 64 rows: no room for the scores
    ("f32", 40, 4, 8, 512, 64, 40, None),                # 160 rows: the larger tiles
    ("bf16", 2, 3, 4, 256, 64, 50, [50, 33]),            # 16-bit storage on this path
    ("f16", 2, 2, 6, 96, 16, 21, [21, 4]),
    # one launch: row tiles of 1 to 4 with and without padding rows, both widths, both head sizes, one position
    ("f32", 3, 16, 4, 64, 16, 31, [31, 16, 1]),
    ("f32", 2, 5, 4, 64, 16, 64, [64, 63]),
    ("f32", 2, 9, 2, 128, 64, 100, [100, 3]),
    ("f32", 2, 16, 2, 128, 64, 97, [97, 96]),
    ("f32", 1, 1, 1, 128, 128, 1, [1]),
    ("f32", 2, 6, 8, 128, 16, 80, [80, 47]),
    ("bf16", 2, 3, 4, 64, 16, 40, [40, 7]),
    ("f16", 2, 4, 2, 128, 64, 33, [33, 32]),
    ("f32", 2, 16, 4, 64, 16, 128, [128, 113]),          # the largest score matrix, and one column more than it holds
    ("f32", 2, 16, 4, 64, 16, 129, [129, 128]),
    ("f32", 2, 4, 4, 128, 32, 256, [256, 241]),          # the same at d_m 128
]


@pytest.mark.parametrize("dtype,B,beam,heads,d_m,d_k,n,lens", CASES)
def test_fp32_arithmetic_path(dtype, B, beam, heads, d_m, d_k, n, lens):
    w = wl.custom(f"f32path_{dtype}_{heads}x{beam}_{d_m}_{n}", dtype=dtype, B=B, beam=beam, heads=heads, d_m=d_m, d_k=d_k,
                  n=n, len_lo=1, len_hi=n, index=90)
    W = wl.weights(w)
    H, Q, L = wl.batch(w, poison=False)
    L = L if lens is None else np.asarray(lens, dtype=np.int32)
    ref = oracle_out(w, W, H, Q, L)
    for b in range(B):
        H[b, L[b]:] = np.nan
    layer = make_layer(w, W)
    assert not layer.uses_mfma
    err = rel_err(gpu_out(layer, w, H, Q, L), ref)
    record(f"{w.name}: err={err:.3e}")
    # 16-bit storage is widened exactly and every product and sum is fp32, so the fp32 bar holds for it as well
    assert err <= TOL["f32"]
    layer.close()


@pytest.mark.parametrize("beam,heads,d_m", [(2, 4, 64), (8, 4, 64), (16, 4, 64), (3, 2, 128), (12, 2, 128)])
def test_one_launch_positions_dealt_to_wavefronts(beam, heads, d_m):
    """The weighted sum of the one-launch step: one, two, four or eight wavefronts with positions of a tile (fewer than there are for
    it, and a number that is no power of two), and a second and third round of positions; with biases and without."""
    wide = 2 * beam * heads <= 32
    n = 128 if not wide else 300 if d_m == 64 else 256
    lens = [16, 17, 47, 81, 128, n]
    w = wl.custom(f"one_launch_{heads}x{beam}_{d_m}", dtype="f32", B=len(lens), beam=beam, heads=heads, d_m=d_m, d_k=d_m // heads, n=n, index=92)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    L = np.asarray(lens, dtype=np.int32)
    for biased in (True, False):
        if not biased:
            W = {k: v if k[0] == "W" else np.zeros_like(v) for k, v in W.items()}
        ref = oracle_out(w, W, H, Q, L)
        Hp = H.copy()
        for b in range(len(lens)):
            Hp[b, L[b]:] = np.nan
        layer = make_layer(w, W if biased else {k: v for k, v in W.items() if k[0] == "W"})
        err = rel_err(gpu_out(layer, w, Hp, Q, L), ref)
        record(f"{w.name}: biased={biased} err={err:.3e}")
        assert err <= TOL["f32"]
        layer.close()


@pytest.mark.parametrize("B,beam,d_m,n", [
    (224, 2, 96, 64),            # scores: 896 workgroups of 16 x 16 outputs, requested early, and four more
    (225, 2, 96, 64),
    (128, 4, 96, 64),            # 512 of 32 x 16, early, and four more
    (129, 4, 96, 64),
    (256, 4, 96, 61),            # 512 of 32 x 32
    (64, 4, 528, 57),            # K >= 512: a whole group of slices, one that is not, and a slice of its own; 32 x 16 outputs
    (32, 16, 528, 64),           # 32 x 32 outputs
])
@pytest.mark.parametrize("off", [0, 1])
def test_forms_of_the_fp32_products(B, beam, d_m, n, off):
    """Both sides of the lines between the forms of the fp32 products, with operands on a 16-byte boundary and one element past it;
    lengths from 1 up, so that most workgroups of a short element have nothing to do."""
    import torch
    w = wl.custom(f"forms_{B}x{beam}_{d_m}_{n}", dtype="f32", B=B, beam=beam, heads=6, d_m=d_m, d_k=d_m // 6, n=n, index=95)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w, poison=False)
    L = np.asarray([1 + (b * 13) % n for b in range(B)], dtype=np.int32)
    ref = oracle_out(w, W, H, Q, L)
    for b in range(B):
        H[b, L[b]:] = np.nan

    def placed(x):
        t = torch.empty(x.size + 4, device="cuda")[off:off + x.size].view(*x.shape)
        t.copy_(torch.from_numpy(x))
        return t
    layer = make_layer(w, W)
    y = layer.decode_step(placed(H), torch.from_numpy(L).cuda(), placed(Q))
    err = rel_err(y.cpu().numpy(), ref)
    record(f"{w.name}: off={off} err={err:.3e}")
    assert not layer.uses_mfma and err <= TOL["f32"]
    layer.close()


@pytest.mark.parametrize("d_m,heads", [(64, 4), (320, 5)])
def test_operands_aligned_to_one_element(d_m, heads):
    """H, queries and out one element past a 16-byte boundary, H with a batch stride that is no multiple of four."""
    import torch
    w = wl.custom(f"unaligned_{d_m}", dtype="f32", B=2, beam=3, heads=heads, d_m=d_m, d_k=d_m // heads, n=45, index=91)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w)
    L = np.asarray([45, 18], dtype=np.int32)
    ref = oracle_out(w, W, H, Q, L)
    stride = w.n * w.d_m + 3
    buf = torch.full((1 + w.B * stride,), float("nan"), device="cuda")
    Hv = torch.as_strided(buf, (w.B, w.n, w.d_m), (stride, w.d_m, 1), 1)
    Hv.copy_(to_device(H, "f32"))
    qbuf = torch.empty(1 + Q.size, device="cuda")
    Qv = qbuf[1:].view(w.B, w.beam, w.d_m)
    Qv.copy_(to_device(Q, "f32"))
    obuf = torch.full((1 + Q.size + 1,), 7.0, device="cuda")
    out = obuf[1:-1].view(w.B, w.beam, w.d_m)
    layer = make_layer(w, W)
    layer.decode_step(Hv, torch.from_numpy(L).cuda(), Qv, out=out)
    torch.cuda.synchronize()
    assert float(obuf[0]) == 7.0 and float(obuf[-1]) == 7.0
    assert rel_err(out.cpu().numpy(), ref) <= TOL["f32"]
    layer.close()


@pytest.mark.parametrize("d_m,heads,beam,n,bound", [(64, 4, 2, 32, 2.6e-7), (64, 4, 3, 200, 2.9e-7), (128, 2, 4, 150, 3.9e-7), (128, 8, 2, 60, 3.9e-7)])
def test_one_launch_step_sums_in_short_chains(d_m, heads, beam, n, bound):
    """Relative 2-norm error of the step against fp64.  m additions one after the other cost about u sqrt(m / 2) of the sum's
    norm (u = 2.4e-8, one rounding's rms): 1.4e-7 for the 64 terms of a product in one chain, 0.7e-7 in four; products follow
    each other four times.  Measured with one chain 3.4e-7 to 5.0e-7, with four 1.9e-7 to 2.7e-7; the bounds lie between."""
    w = wl.custom(f"chains_{d_m}_{heads}", dtype="f32", B=16, beam=beam, heads=heads, d_m=d_m, d_k=d_m // heads, n=n, len_lo=(n + 1) // 2,
                  len_hi=n, index=92)
    W = wl.weights(w)
    H, Q, L = wl.batch(w, poison=False)
    rep = err_report(gpu_out(make_layer(w, W), w, H, Q, L), oracle_out(w, W, H, Q, L))
    record(f"{w.name}: {fmt_report(rep)}")
    assert rep["l2"] <= bound


@pytest.mark.parametrize("d_m,heads,timed", [(64, 4, 0), (256, 4, 3)])
def test_core_timing_reports_attention_cores_only(d_m, heads, timed):
    """A step that runs as one launch has no core kernel (a3-a5) to bracket: it must not report its own time as the core's."""
    w = wl.custom(f"timing_{d_m}", dtype="f32", B=2, beam=2, heads=heads, d_m=d_m, d_k=d_m // heads, n=32, index=93)
    layer = make_layer(w, wl.weights(w))
    H, Q, L = wl.batch(w)
    layer.core_timing(8)
    for _ in range(3):
        gpu_out(layer, w, H, Q, L)
    ms = layer.read_core_timing(8)
    assert len(ms) == timed and all(t > 0.0 for t in ms)
    layer.close()


KEY_RANGE_CASES = [
    # dtype, B, heads, beam, d_m, n, splits: R x n beyond 8 x R64 x d_m, so no room for the scores
    ("f16", 2, 4, 16, 64, 516, 0),               # one element past the line, eight ranges
    ("bf16", 3, 16, 4, 320, 2570, 0),            # two columns per thread, a length that is no multiple of four
    ("f32", 1, 16, 4, 640, 5124, 3),             # three columns per thread in use of four; ranges by request
    ("bf16", 2, 2, 32, 64, 700, 1),              # one range: nothing to merge
    ("f32", 2, 4, 16, 64, 520, 15),              # more ranges than the partials' room: eight
    ("f16", 1, 13, 5, 1040, 16420, 0),           # R64 of 128 for 65 rows; eight columns per thread
]


def _key_range_inputs(dtype, B, heads, beam, d_m, n):
    R = heads * beam
    assert R * ((n + 3) // 4 * 4) > 8 * ((R + 63) // 64 * 64) * d_m
    w = wl.custom(f"ranges_{dtype}_{d_m}_{n}", dtype=dtype, B=B, beam=beam, heads=heads, d_m=d_m, d_k=d_m // heads, n=n, index=94)
    W = wl.weights(w)
    H, Q, _ = wl.batch(w)
    L = np.asarray([n, n // 2 + 1, 7][:B], dtype=np.int32)
    return w, W, H, Q, L


@pytest.mark.parametrize("dtype,B,heads,beam,d_m,n,splits", KEY_RANGE_CASES)
def test_keys_too_long_for_scores_in_memory(dtype, B, heads, beam, d_m, n, splits):
    """The key-range core and its merge, against the oracle's own Eq. 9 order (fp64): H is not projected, which at these
    lengths is most of the work."""
    w, W, H, Q, L = _key_range_inputs(dtype, B, heads, beam, d_m, n)
    ref = oracle.el_reference(H, L, Q, W["Wq"], W["bq"], W["Wk"], W["bk"], W["Wv"], W["bv"], W["Wo"], W["bo"], heads=heads, d_k=w.d_k)
    for b in range(B):
        H[b, L[b]:] = np.nan
    layer = make_layer(w, W)
    layer.set_splits(splits)
    err = rel_err(gpu_out(layer, w, H, Q, L), ref)
    record(f"{w.name} splits={splits}: err={err:.3e}")
    assert not layer.uses_mfma and err <= TOL["f32"]
    layer.close()
