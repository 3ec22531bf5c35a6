"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded inputs.

Bar (stated by the benchmark spec): segment index k, LUT index l0, the domain predicate In(x) and the integer
codes bit-exact; outputs within |dy| <= 1e-5 * sum_i |phi_ij(x_i)| + 1e-6 (fp32).  The interpolation weight w is
produced by the same IEEE fp32 operations on both sides and is compared bit-exactly as well.
"""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
from lutkan_inputs import (ASYM_UINT8, CLIP_X, CLOSED, HALF_OPEN, SYM_INT8, ZERO_SPLINE, case_a, cfg1, cfg2, cfg3, cfg4,
                           cfg5, random_layer)
from lutkan_inputs import per_input_layer

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2601_03332_amd as lk  # noqa: E402

DEV = "cuda:0"
RTOL, ATOL = 1e-5, 1e-6


def _say(msg):
    print(msg, flush=True)


_COMPILED = {}


def _compile_both(s, param_fp16=False):
    """Library artifact + oracle artifact for a layer spec; the codes must already agree bit for bit.
    Cached per table content (the contract fields do not change the tables)."""
    key = (s.d, s.m, s.G, s.L, s.scheme, hash(s.coef.tobytes()), hash(s.ext_knots.tobytes()), param_fp16, s.per_input,
           None if s.edge_scales is None else hash(b"".join(a.tobytes() for a in s.edge_scales)))
    if key not in _COMPILED:
        if len(_COMPILED) > 4:
            _COMPILED.clear()
        art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob,
                                edge_scales=s.edge_scales, param_dtype=lk.PARAM_FP16 if param_fp16 else lk.PARAM_FP32,
                                knots_per_input=s.per_input)
        ora = oracle.compile_layer(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, param_fp16=param_fp16,
                                   per_input=s.per_input)
        assert np.array_equal(art.q, ora.q) and np.array_equal(art.scale, ora.scale) and np.array_equal(art.y_min, ora.y_min)
        _COMPILED[key] = (art, ora)
    return _COMPILED[key]


def _device_layer(art, s, algo=lk.ALGO_AUTO, wide=None):
    return art.to_device(DEV, algo, wide=wide).with_contract(s.boundary, s.oob)


def _assert_close(y_gpu, ref, what):
    err = np.abs(y_gpu.astype(np.float64) - ref.y.astype(np.float64))
    tol = RTOL * ref.A + ATOL
    nan_ok = np.isnan(y_gpu) == np.isnan(ref.y)
    assert nan_ok.all(), f"{what}: NaN pattern differs"
    bad = np.nan_to_num(err, nan=0.0) > np.nan_to_num(tol, nan=np.inf)
    assert not bad.any(), f"{what}: {bad.sum()} outputs out of tolerance, worst ratio {np.nanmax(err / tol):.3g}"
    return float(np.nanmax(err / tol))


def _check_layer(s, x, algo, codes=False, what="", param_fp16=False, wide=None):
    art, ora = _compile_both(s, param_fp16)
    layer = _device_layer(art, s, algo, wide)
    xg = torch.from_numpy(x).to(DEV)
    _say(f"case {what} d={s.d} m={s.m} K={s.G} L={s.L} scheme={s.scheme} boundary={s.boundary} oob={s.oob} "
         f"B={x.shape[0]} algo={algo} jt={art.info.jt} param_fp16={param_fp16} wide={wide}")
    y, k, l0, inside, w, q01 = lk.lutkan_forward_trace(layer, xg, codes=codes)
    stats = torch.zeros(2, dtype=torch.int64, device=DEV)
    y2 = lk.lutkan_forward(layer, xg, stats=stats)
    torch.cuda.synchronize()
    ref = oracle.lut_forward(ora, s.boundary, s.oob, x, trace=True, codes=codes, edge_scalars=s.edge_scales)
    np.testing.assert_array_equal(k.cpu().numpy(), ref.k)
    np.testing.assert_array_equal(l0.cpu().numpy(), ref.l0)
    np.testing.assert_array_equal(inside.cpu().numpy(), ref.inside)
    np.testing.assert_array_equal(w.cpu().numpy().view(np.uint32), ref.w.view(np.uint32))
    if codes:
        np.testing.assert_array_equal(q01.cpu().numpy(), ref.q01)
    worst = _assert_close(y.cpu().numpy(), ref, what)
    worst = max(worst, _assert_close(y2.cpu().numpy(), ref, what + " (plain launch)"))
    if not codes and algo != lk.ALGO_AUTO:              # a named kernel: trace and plain launch are the same arithmetic
        assert torch.equal(y, y2) or np.array_equal(np.isnan(y.cpu().numpy()), np.isnan(y2.cpu().numpy()))
    st = stats.cpu().numpy()
    assert (int(st[0]), int(st[1])) == (ref.oob_count, ref.oob_any_rows)
    return worst


def test_cfg1_tiny_layer_with_codes():
    w = cfg1()
    _check_layer(w.layers[0], w.x, lk.ALGO_GATHER, codes=True, what=w.name)


PROPERTY_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B, uniform
    (101, 1, 1, 3, 2, SYM_INT8, CLOSED, CLIP_X, 1, True),
    (102, 1, 5, 5, 16, ASYM_UINT8, HALF_OPEN, CLIP_X, 33, False),
    (103, 7, 1, 4, 32, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 257, True),
    (104, 5, 3, 6, 33, ASYM_UINT8, CLOSED, ZERO_SPLINE, 100, False),
    (105, 13, 17, 11, 64, SYM_INT8, CLOSED, CLIP_X, 513, False),
    (106, 9, 70, 5, 128, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 65, True),
    (107, 3, 130, 8, 16, SYM_INT8, HALF_OPEN, CLIP_X, 31, False),
    (108, 20, 64, 5, 64, ASYM_UINT8, CLOSED, CLIP_X, 300, True),
    (109, 6, 200, 64, 8, SYM_INT8, CLOSED, ZERO_SPLINE, 129, False),
    (110, 70, 2, 5, 64, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 5000, True),     # inputs split into chunks, 4-column tile
    (111, 130, 9, 7, 32, SYM_INT8, CLOSED, CLIP_X, 3001, False),            # 16-column tile, 8 chunks
    (112, 33, 30, 9, 16, SYM_INT8, HALF_OPEN, CLIP_X, 40000, True),         # 32-column tile, many row tiles
]


@pytest.mark.parametrize("case", PROPERTY_CASES, ids=lambda c: f"seed{c[0]}")
def test_property_layers_gather_with_codes(case):
    seed, d, m, G, L, scheme, boundary, oob, B, uniform = case
    w = random_layer(seed, d, m, G, L, scheme, boundary, oob, B, uniform=uniform)
    _check_layer(w.layers[0], w.x, lk.ALGO_GATHER, codes=(B * d * m <= 2_000_000), what=w.name)
    _check_layer(w.layers[0], w.x, lk.ALGO_TILED, what=w.name)          # narrow column tiles: 4..64 columns


TILED_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B
    (201, 17, 128, 5, 32, SYM_INT8, CLOSED, CLIP_X, 700),
    (202, 33, 130, 8, 64, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 1025),
    (203, 5, 70, 10, 64, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 64),
    (204, 40, 300, 6, 16, ASYM_UINT8, CLOSED, CLIP_X, 4099),
    (205, 64, 256, 8, 128, SYM_INT8, CLOSED, ZERO_SPLINE, 2500),     # slice too big for 128-wide tiles -> 64-wide
    (206, 64, 256, 8, 128, ASYM_UINT8, HALF_OPEN, CLIP_X, 9000),
    (207, 3, 1000, 10, 64, SYM_INT8, CLOSED, CLIP_X, 20000),         # enough rows for the 32-rows-per-wave variant
    (208, 1, 128, 2, 2, ASYM_UINT8, CLOSED, CLIP_X, 1),
    (209, 7, 70, 16, 128, SYM_INT8, CLOSED, CLIP_X, 1500),           # 2048 table rows: 16-column tiles of a wide layer
    (210, 5, 50, 32, 128, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 2100), # 4096 table rows: 8-column tiles, ragged last tile
    (211, 3, 21, 64, 200, SYM_INT8, HALF_OPEN, CLIP_X, 300),         # 12800 table rows: 4-column tiles
    (213, 5000, 4, 3, 8, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 50),    # very many inputs: 79 locate tiles, many chunks
    (214, 2, 5000, 3, 8, SYM_INT8, CLOSED, CLIP_X, 33),              # very many outputs: 40 column tiles
]


@pytest.mark.parametrize("case", TILED_CASES, ids=lambda c: f"seed{c[0]}")
def test_property_layers_tiled(case):
    seed, d, m, G, L, scheme, boundary, oob, B = case
    w = random_layer(seed, d, m, G, L, scheme, boundary, oob, B, uniform=(seed % 2 == 0))
    _check_layer(w.layers[0], w.x, lk.ALGO_TILED, what=w.name)
    _check_layer(w.layers[0], w.x, lk.ALGO_GATHER, what=w.name)


WIDE_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B, with_base     64-column tiles whose wide slice (2 bytes per code) fits the LDS twice
    (701, 17, 128, 5, 32, SYM_INT8, CLOSED, CLIP_X, 700, False),
    (702, 33, 130, 8, 64, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 1025, False),     # 514 code rows: the largest wide slices; ragged last tile
    (703, 64, 256, 8, 64, SYM_INT8, CLOSED, ZERO_SPLINE, 2500, False),
    (704, 40, 300, 6, 16, ASYM_UINT8, CLOSED, CLIP_X, 4099, False),
    (705, 1, 64, 2, 2, ASYM_UINT8, CLOSED, CLIP_X, 1, False),
    (706, 300, 64, 5, 32, SYM_INT8, HALF_OPEN, CLIP_X, 9000, False),            # many inputs: chunks and the summing pass
    (707, 3, 1000, 10, 50, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 20000, False),     # 16 column tiles, three slice buffers
    (708, 64, 128, 5, 32, ASYM_UINT8, CLOSED, CLIP_X, 70000, True),             # spline_component: base branch as a product, 8-byte records
    (709, 24, 70, 6, 16, SYM_INT8, CLOSED, ZERO_SPLINE, 3000, True),            # spline_component with 16-byte records: byte form or fp32 values
    (713, 40, 128, 5, 32, ASYM_UINT8, HALF_OPEN, CLIP_X, 20000, True),          # the same at 16 row steps per wave
    (710, 64, 256, 8, 32, SYM_INT8, HALF_OPEN, CLIP_X, 16384 + 3, False),       # large enough for the launch planning to pick the wide form
    (711, 20, 192, 5, 32, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 5001, False),     # masked inputs on a layer that has both wide forms
    (712, 96, 64, 3, 90, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 33000, False),       # 272 value rows: the largest fp32 slices (two buffers)
]


@pytest.mark.parametrize("cb", [2, 4], ids=["binary16_codes", "fp32_values"])
@pytest.mark.parametrize("case", WIDE_CASES, ids=lambda c: f"seed{c[0]}")
def test_wide_table_form(case, cb):
    """The wide forms of the device table against the oracle, to the bar of every other path.  16-bit codes (no byte
    unpacking in the tiled kernel): the arithmetic after the unpacking is that of the byte form, so with the same launch
    plan the outputs agree bit for bit.  fp32 values (Eq. 10 applied when the table is built, the kernel interpolates
    the values): a different rounding order, so only the oracle is the measure."""
    seed, d, m, G, L, scheme, boundary, oob, B, with_base = case
    w = random_layer(seed, d, m, G, L, scheme, boundary, oob, B, uniform=(seed % 2 == 0), oob_frac=0.3, with_base=with_base)
    s = w.layers[0]
    x = w.x.copy()
    if B > 1:
        x[B // 2, d // 3] = np.nan
    art, ora = _compile_both(s)
    assert art.info.jt == 64
    value_rows_fit = (art.info.K * L + 2 + with_base) * 256 <= 72 * 1024
    if cb == 4 and not value_rows_fit:
        with pytest.raises(lk.LutKanError) as e:
            art.to_device(DEV, wide=4)
        assert "no wide table form of 4 bytes" in str(e.value)
        assert art.to_device(DEV, wide=True).c.wide_code_bytes == 2           # "any": the form the layer has
        return
    wide, byte = _device_layer(art, s, lk.ALGO_TILED_WIDE, wide=cb), _device_layer(art, s, lk.ALGO_TILED, wide=False)
    assert wide.wide_table is not None and byte.wide_table is None and wide.c.wide_code_bytes == cb
    if cb == 2:
        assert wide.wide_table.numel() == art.info.table_bytes + art.info.n_tiles * d * (art.info.K * L + 2) * 64
    else:
        assert wide.wide_table.numel() == art.info.n_tiles * d * (art.info.K * L + 2 + with_base) * 256
        assert art.to_device(DEV, wide=True).c.wide_code_bytes == 4
    xg = torch.from_numpy(x).to(DEV)
    if with_base and B * d * m < 5e8 and cb == 2:
        # 16-byte records (the base branch inside the edge kernel) go with the byte form or with fp32 values
        with pytest.raises(lk.LutKanError) as e:
            lk.lutkan_forward(wide, xg)
        assert str(e.value).startswith("[-5]") and "16-byte records" in str(e.value)
        _check_layer(s, x, lk.ALGO_TILED, what=w.name + " (wide table present, byte form runs)", wide=cb)
        assert "tiled np=" in lk.lutkan_last_plan()
        return
    tag = "tiled wide np=" if cb == 2 else "tiled wide32 np="
    worst = _check_layer(s, x, lk.ALGO_TILED_WIDE, what=w.name + f" (wide form, {cb} bytes per code)", wide=cb)
    y_wide = lk.lutkan_forward(wide, xg)
    plan_wide = lk.lutkan_last_plan()
    y_byte = lk.lutkan_forward(byte, xg)
    plan_byte = lk.lutkan_last_plan()
    _say(f"wide: {plan_wide!r}  byte: {plan_byte!r}  worst error / tolerance {worst:.3g}")
    assert tag in plan_wide and " wide" not in plan_byte
    if cb == 2 and plan_wide.replace("tiled wide", "tiled") == plan_byte:
        assert bool(((y_wide == y_byte) | (torch.isnan(y_wide) & torch.isnan(y_byte))).all())
    # the two phases apart, and the entry point with the built-in scratch, take the same form
    ws = torch.empty(lk.lutkan_forward_workspace_bytes(wide, B), dtype=torch.uint8, device=DEV)
    lk.lutkan_forward_locate(wide, xg, ws)
    y_two = lk.lutkan_forward_edges(wide, B, torch.full((B, m), 3.0, dtype=torch.float32, device=DEV), ws)
    assert bool(((y_two == y_wide) | (torch.isnan(y_two) & torch.isnan(y_wide))).all())
    if lk.lutkan_forward_workspace_bytes(wide, B) <= lk.STATIC_SCRATCH_BYTES:
        y_static = lk.lutkan_forward_static_scratch(wide, xg, torch.full((B, m), -3.0, dtype=torch.float32, device=DEV))
        assert bool(((y_static == y_wide) | (torch.isnan(y_static) & torch.isnan(y_wide))).all())
    # left to the launch planning: 16-bit codes run on large batches of symmetric layers, fp32 values with both schemes
    auto = _device_layer(art, s, lk.ALGO_AUTO, wide=cb)
    lk.lutkan_forward(auto, xg)
    if cb == 2 and scheme == ASYM_UINT8:
        assert " wide" not in lk.lutkan_last_plan(), lk.lutkan_last_plan()
    elif B * d * m >= 2e8:
        assert tag in lk.lutkan_last_plan(), lk.lutkan_last_plan()
    # the default upload: fp32 values where they fit, else 16-bit codes for symmetric layers; layers of some size only
    default = art.to_device(DEV).c.wide_code_bytes
    assert default == (0 if d * m < 4096 else 4 if value_rows_fit else 2 if scheme == SYM_INT8 else 0)


def test_wide_table_form_exists_only_where_it_pays():
    """No wide form on tiles narrower than 64 columns or when two wide slices do not fit the LDS (the widest layer:
    642 code rows); asking for one is an error, the default upload simply goes without."""
    for d, m, G, L in ((8, 32, 5, 16), (4, 1024, 10, 64), (4, 256, 8, 128)):
        w = random_layer(720, d, m, G, L, SYM_INT8, CLOSED, CLIP_X, 8)
        art, _ = _compile_both(w.layers[0])
        assert art.to_device(DEV).wide_table is None
        with pytest.raises(lk.LutKanError):
            art.to_device(DEV, wide=True)


@pytest.mark.parametrize("case", [(731, 5, 130, 6, 16, SYM_INT8, False), (732, 3, 64, 5, 32, ASYM_UINT8, False),
                                  (733, 4, 200, 8, 8, ASYM_UINT8, True), (734, 2, 70, 4, 64, SYM_INT8, True)],
                         ids=lambda c: f"seed{c[0]}")
def test_wide_tables_hold_exactly_what_the_codes_stand_for(case):
    """The two wide forms as built on the device, read back and compared bit for bit with what the oracle's artifact
    arrays say they must hold: the binary16 pattern of q * 2^-24 (sign and magnitude) resp. the fp32 value of Eq. 10,
    fl(y_min + fl(alpha * q)), for every (tile, input, code row, column); the two rows after the last code row and
    the columns past m are zero."""
    seed, d, m, G, L, scheme, half = case
    w = random_layer(seed, d, m, G, L, scheme, CLOSED, CLIP_X, 4)
    s = w.layers[0]
    art, ora = _compile_both(s, param_fp16=half)
    K, jt, n_tiles = art.info.K, art.info.jt, art.info.n_tiles
    assert jt == 64 and K == ora.K
    rows = K * L + 2
    q = ora.q.reshape(d, m, K * L).astype(np.int32)                  # [i][j][row]
    alpha = np.repeat(ora.scale.reshape(d, m, K), L, axis=2)         # the parameters of each row's segment
    y_min = np.repeat(ora.y_min.reshape(d, m, K), L, axis=2)
    values = (y_min + (alpha * q.astype(np.float32)).astype(np.float32)).astype(np.float32)        # two fp32 roundings
    bits16 = np.where(q < 0, 0x8000 | -q, q).astype(np.uint16)
    _say(f"case {w.name} wide table contents, param_fp16={half}")
    for cb, want, dtype in ((2, bits16, np.uint16), (4, values, np.float32)):
        layer = art.to_device(DEV, wide=cb)
        blob = layer.c.wide_blob_bytes
        host = layer.wide_table.cpu().numpy().reshape(n_tiles, d, blob)
        codes_off = blob - (-(-rows * jt * cb // 16) * 16)             # the code rows end the slice (padded to 16 bytes)
        if cb == 4:
            assert codes_off == 0                                    # phi layer: no base row, no parameter rows
        got = np.ascontiguousarray(host[:, :, codes_off:codes_off + rows * jt * cb]).view(dtype).reshape(n_tiles, d, rows, jt)
        full = np.zeros((n_tiles * jt, d, rows), dtype=dtype)
        full[:m, :, :K * L] = np.transpose(want, (1, 0, 2))          # [j][i][row]
        expect = np.transpose(full.reshape(n_tiles, jt, d, rows), (0, 2, 3, 1))                   # [t][i][row][column]
        if cb == 4:
            assert np.array_equal(got, expect)                       # (padding: 0 * -128 under y_min = 0 is +0)
        else:
            pad = np.zeros(expect.shape, dtype=bool)
            pad[:, :, K * L:, :] = True
            pad |= (np.arange(n_tiles * jt).reshape(n_tiles, jt) >= m)[:, None, None, :]
            assert np.array_equal(got[~pad], expect[~pad])
            # padding holds a code byte of 0 or the code 0 (excess-128: byte 0 reads as -128, under alpha = 0)
            assert np.isin(got[pad], (0, 0x8080)).all()
        if cb == 2:                                                  # everything before the code rows is the byte table's
            byte = np.asarray(art.table).reshape(n_tiles, d, art.info.blob_bytes)
            assert np.array_equal(host[:, :, :codes_off], byte[:, :, :codes_off])


@pytest.mark.parametrize("base", [False, True], ids=["phi", "spline_component"])
def test_largest_slices_with_the_largest_record_buffers_fill_the_lds(base):
    """The LDS budget at its edge: 64-column slices of 72 KiB (64 KiB with the base branch, whose records are 16 bytes)
    at a batch large enough for 16 row steps per wave, so that two slice buffers and the record buffers take all but
    a few hundred bytes of the 160 KiB of a compute unit.  Sampled rows against the oracle."""
    L = 122 if base else 139         # 8 L + 2 code rows of 64 bytes + parameters: just under the budget
    B = 262144 + 3
    w = random_layer(230 + base, 4, 64, 8, L, SYM_INT8, HALF_OPEN, ZERO_SPLINE, B, with_base=base)
    s = w.layers[0]
    art, ora = _compile_both(s)
    budget = (64 if base else 72) * 1024
    assert art.info.jt == 64 and budget - 1024 < art.info.blob_bytes <= budget
    layer = _device_layer(art, s)
    xg = torch.from_numpy(w.x).to(DEV)
    _say(f"case {w.name} B={B} slice of {art.info.blob_bytes} bytes")
    y = lk.lutkan_forward(layer, xg)
    assert lk.lutkan_last_plan().startswith("locate; tiled np=16 "), lk.lutkan_last_plan()
    lds = 2 * art.info.blob_bytes + 16 * 2 * 64 * (16 if base else 8)
    assert 160 * 1024 - 1024 < lds <= 160 * 1024
    rows = np.unique(np.concatenate([np.random.Generator(np.random.PCG64(5)).integers(0, B, size=1500), [0, B - 1]]))
    ref = oracle.lut_forward(ora, s.boundary, s.oob, w.x[rows], edge_scalars=s.edge_scales)
    _assert_close(y[torch.from_numpy(rows).to(DEV)].cpu().numpy(), ref, w.name)


def test_table_too_large_for_any_tile_runs_on_the_gather_kernel():
    """32768 table rows: not even a 4-column slice fits the LDS budget; AUTO takes the gather kernel on 32-column
    tiles, and asking for the tiled kernel is an error, not a silent fallback."""
    w = random_layer(212, 2, 40, 64, 512, ASYM_UINT8, CLOSED, ZERO_SPLINE, 257)
    s = w.layers[0]
    _check_layer(s, w.x, lk.ALGO_AUTO, what=w.name)
    art = _compile_both(s)[0]
    assert art.info.jt == 32 and art.info.blob_bytes > 72 * 1024
    with pytest.raises(lk.LutKanError) as e:
        lk.lutkan_forward(_device_layer(art, s, lk.ALGO_TILED), torch.from_numpy(w.x).to(DEV))
    assert str(e.value).startswith("[-5]")


FP16_PARAM_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B          float16 scale / y_min (Sec. 4.6)
    (601, 4, 3, 5, 16, SYM_INT8, CLOSED, CLIP_X, 200),                # 4-column tile
    (602, 78, 16, 5, 64, ASYM_UINT8, CLOSED, CLIP_X, 3000),           # 16-column tile, inputs split
    (603, 33, 130, 8, 64, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 1025),  # 128-column tiles, ragged last tile
    (604, 64, 256, 8, 128, SYM_INT8, CLOSED, ZERO_SPLINE, 2500),      # 64-column tiles
    (605, 40, 300, 6, 16, SYM_INT8, HALF_OPEN, CLIP_X, 4099),
    (606, 20, 64, 10, 64, ASYM_UINT8, CLOSED, CLIP_X, 17000),         # 16 row steps per wave
]


@pytest.mark.parametrize("case", FP16_PARAM_CASES, ids=lambda c: f"seed{c[0]}")
def test_fp16_parameters(case):
    seed, d, m, G, L, scheme, boundary, oob, B = case
    w = random_layer(seed, d, m, G, L, scheme, boundary, oob, B, uniform=(seed % 2 == 0))
    _check_layer(w.layers[0], w.x, lk.ALGO_TILED, what=w.name, param_fp16=True)
    _check_layer(w.layers[0], w.x, lk.ALGO_GATHER, codes=(B * d * m <= 2_000_000), what=w.name, param_fp16=True)


@pytest.mark.parametrize("case", FP16_PARAM_CASES, ids=lambda c: f"seed{c[0]}")
def test_fp16_parameters_with_spline_component(case):
    """The deployment combination of Sec. 8: asymmetric or symmetric codes, float16 scale / y_min, Eq. 2's base branch
    and per-edge scalars; the scalars multiply the dequantised value, the parameters stay the rounded ones."""
    seed, d, m, G, L, scheme, boundary, oob, B = case
    w = random_layer(seed + 50, d, m, G, L, scheme, boundary, oob, B, uniform=(seed % 2 == 1), with_base=True)
    _check_layer(w.layers[0], w.x, lk.ALGO_TILED, what=w.name, param_fp16=True)
    _check_layer(w.layers[0], w.x, lk.ALGO_GATHER, codes=(B * d * m <= 2_000_000), what=w.name, param_fp16=True)


PER_INPUT_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B, with_base, param_fp16
    (801, 1, 1, 3, 2, SYM_INT8, CLOSED, CLIP_X, 1, False, False),
    (802, 3, 5, 5, 16, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 300, False, False),      # 16 inputs per locate block
    (803, 20, 16, 8, 64, SYM_INT8, HALF_OPEN, CLIP_X, 1025, True, False),           # 32 inputs per locate block
    (804, 70, 130, 10, 32, ASYM_UINT8, CLOSED, ZERO_SPLINE, 2100, False, True),     # two blocks of 64 inputs, ragged
    (805, 33, 64, 64, 8, SYM_INT8, CLOSED, CLIP_X, 700, True, True),                # the longest knot vectors
    (806, 129, 40, 6, 128, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 4099, True, False),
]


@pytest.mark.parametrize("case", PER_INPUT_CASES, ids=lambda c: f"seed{c[0]}")
def test_one_knot_vector_per_input(case):
    """Sec. 6.2's knot grid "shared per input dimension": every input is located, clipped and masked on its own knot
    vector (different domains, uniform and non-uniform); LUT layer (both kernels, counters) and B-spline layer."""
    seed, d, m, G, L, scheme, boundary, oob, B, with_base, half = case
    w = per_input_layer(seed, d, m, G, L, scheme, boundary, oob, B, with_base=with_base)
    s = w.layers[0]
    _check_layer(s, w.x, lk.ALGO_AUTO, what=w.name, param_fp16=half)
    _check_layer(s, w.x, lk.ALGO_GATHER, codes=(B * d * m <= 2_000_000), what=w.name, param_fp16=half)
    art = _compile_both(s, half)[0]
    xg = torch.from_numpy(w.x).to(DEV)
    refb = oracle.bspline_forward(d, m, G, s.p, s.ext_knots, s.coef, boundary, oob, w.x, edge_scalars=s.edge_scales, per_input=True)
    for algo in (lk.ALGO_AUTO, lk.ALGO_GATHER):
        yb = lk.bspline_kan_forward(art.bspline_to_device(DEV, algo), xg)
        torch.cuda.synchronize()
        _assert_close(yb.cpu().numpy(), refb, f"{w.name} bspline algo={algo}")
    # the error statistics with every input's own domain
    y_lut = lk.lutkan_forward(_device_layer(art, s), xg)
    dom = torch.from_numpy(np.ascontiguousarray(art.knots[:, [0, -1]])).to(DEV)
    got = lk.lutkan_error_stats(y_lut, yb, xg, 0.0, 0.0, boundary, input_domain=dom)
    want = oracle.error_stats(y_lut.cpu().numpy(), yb.cpu().numpy(), w.x, art.knots[:, 0], art.knots[:, -1], boundary)
    _same_error_summary(got, want)


def test_per_input_layer_without_its_knot_table_is_refused():
    w = per_input_layer(810, 4, 4, 5, 8, SYM_INT8, CLOSED, CLIP_X, 16)
    s = w.layers[0]
    art = _compile_both(s)[0]
    layer, bl = art.to_device(DEV), art.bspline_to_device(DEV)
    layer.c.input_knots = None
    bl.c.input_ext_knots = None
    xg = torch.from_numpy(w.x).to(DEV)
    for call in (lambda: lk.lutkan_forward(layer, xg), lambda: lk.bspline_kan_forward(bl, xg)):
        with pytest.raises(lk.LutKanError) as e:
            call()
        assert str(e.value).startswith("[-1]")


def test_loaded_artifact_runs_like_the_compiled_one(tmp_path):
    """An artifact written to NPZ + manifest and read back (Sec. 4.6) gives bit-identical outputs and counters."""
    w = random_layer(611, 20, 150, 6, 32, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 3000)
    s = w.layers[0]
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob)
    path = str(tmp_path / "layer.npz")
    art.save(path)
    back = lk.lutkan_artifact_load(path)
    xg = torch.from_numpy(w.x).to(DEV)
    _say(f"case {w.name} loaded artifact jt={back.info.jt}")
    st1, st2 = torch.zeros(2, dtype=torch.int64, device=DEV), torch.zeros(2, dtype=torch.int64, device=DEV)
    y1 = lk.lutkan_forward(art.to_device(DEV), xg, stats=st1)
    y2 = lk.lutkan_forward(back.to_device(DEV), xg, stats=st2)
    torch.cuda.synchronize()
    assert torch.equal(y1, y2) and torch.equal(st1, st2)
    ora = oracle.compile_layer(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme)
    _assert_close(y2.cpu().numpy(), oracle.lut_forward(ora, s.boundary, s.oob, w.x), w.name)


EXTENDED_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B, uniform          LUT and B-spline layer over the extended knot vector
    (801, 3, 5, 5, 16, SYM_INT8, CLOSED, CLIP_X, 300, True),
    (802, 10, 130, 4, 32, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 1500, False),
    (803, 20, 64, 8, 64, SYM_INT8, CLOSED, ZERO_SPLINE, 2000, False),
    (804, 7, 9, 1, 8, ASYM_UINT8, HALF_OPEN, CLIP_X, 500, True),       # one grid interval: R = 4 coefficients
    (805, 5, 40, 58, 4, SYM_INT8, CLOSED, CLIP_X, 700, True),         # K = 64 segments
]


@pytest.mark.parametrize("case", EXTENDED_CASES, ids=lambda c: f"seed{c[0]}")
def test_extended_knot_span(case):
    seed, d, m, G, L, scheme, boundary, oob, B, uniform = case
    w = random_layer(seed, d, m, G, L, scheme, boundary, oob, B, uniform=uniform)
    s = w.layers[0]
    tau = s.ext_knots
    rng = np.random.Generator(np.random.PCG64(seed))
    span = float(tau[-1] - tau[0])
    x = rng.uniform(tau[0] - 0.1 * span, tau[-1] + 0.1 * span, size=(B, d)).astype(np.float32)
    pick = rng.integers(0, B * d, size=B * d // 8)                    # exact extended knots and their neighbours
    vals = tau[rng.integers(0, tau.size, size=pick.size)]
    nudge = rng.integers(-1, 2, size=pick.size)
    x.reshape(-1)[pick] = np.where(nudge < 0, np.nextafter(vals, np.float32(-np.inf)),
                                   np.where(nudge > 0, np.nextafter(vals, np.float32(np.inf)), vals)).astype(np.float32)
    art = lk.lutkan_compile(d, m, G, 3, tau, s.coef, L, scheme, boundary, oob, knot_span=lk.SPAN_EXTENDED)
    ora = oracle.compile_layer(d, m, G, 3, tau, s.coef, L, scheme, extended=True)
    assert np.array_equal(art.q, ora.q) and np.array_equal(art.scale, ora.scale) and np.array_equal(art.y_min, ora.y_min)
    xg = torch.from_numpy(x).to(DEV)
    _say(f"case extended {w.name} K={art.info.K} jt={art.info.jt}")
    y, k, l0, inside, wgt, _ = lk.lutkan_forward_trace(art.to_device(DEV), xg)
    yb = lk.bspline_kan_forward(art.bspline_to_device(DEV), xg)
    yb_g = lk.bspline_kan_forward(art.bspline_to_device(DEV, lk.ALGO_GATHER), xg)
    torch.cuda.synchronize()
    ref = oracle.lut_forward(ora, boundary, oob, x, trace=True)
    np.testing.assert_array_equal(k.cpu().numpy(), ref.k)
    np.testing.assert_array_equal(l0.cpu().numpy(), ref.l0)
    np.testing.assert_array_equal(inside.cpu().numpy(), ref.inside)
    np.testing.assert_array_equal(wgt.cpu().numpy().view(np.uint32), ref.w.view(np.uint32))
    _assert_close(y.cpu().numpy(), ref, w.name)
    refb = oracle.bspline_forward(d, m, G, 3, tau, s.coef, boundary, oob, x, extended=True)
    _assert_close(yb.cpu().numpy(), refb, w.name + " bspline")
    _assert_close(yb_g.cpu().numpy(), refb, w.name + " bspline gather")


def test_special_inputs_nan_inf_all_oob():
    w = random_layer(301, 6, 140, 5, 32, ASYM_UINT8, CLOSED, ZERO_SPLINE, 40)
    x = w.x.copy()
    x[3, 2] = np.nan
    x[5, :] = np.inf
    x[6, :] = -np.inf
    x[7, :] = 1e30
    x[8, 0] = -0.0
    for algo in (lk.ALGO_GATHER, lk.ALGO_TILED):
        for boundary in (HALF_OPEN, CLOSED):
            for oob in (CLIP_X, ZERO_SPLINE):
                s = w.layers[0]
                s.boundary, s.oob = boundary, oob
                _check_layer(s, x, algo, what="special")


def test_domain_ends_at_zero_and_below_and_subnormal_inputs():
    """The safe upper clip value of Eq. 13 in half-open mode is nextafter(t_K, -inf): below t_K = 0 that is the
    smallest negative subnormal, below a negative t_K the next float of larger magnitude.  Shared knots (clip value
    from the host) and one vector per input (clip value computed in the kernel), inputs on and around those values."""
    from lutkan_inputs import LayerSpec, uniform_ext_knots
    rng = np.random.Generator(np.random.PCG64(31))
    G, L, m = 4, 16, 5
    tiny = np.float32(1e-45)                                            # the smallest positive subnormal
    ends = [(-2.0, 0.0), (-3.0, -1.0), (0.0, 2.0), (-1.0, 1.0)]
    specials = []
    for lo, hi in ends:
        for v in (lo, hi):
            v = np.float32(v)
            specials += [v, np.nextafter(v, np.float32(-np.inf)), np.nextafter(v, np.float32(np.inf))]
    specials += [np.float32(0.0), np.float32(-0.0), tiny, -tiny, np.float32(1e-39), np.float32(-1e-39)]
    specials = np.array(specials, dtype=np.float32)
    for boundary in (HALF_OPEN, CLOSED):
        for oob in (CLIP_X, ZERO_SPLINE):
            # one vector per input: the four domains side by side, every special value in every column
            tau = np.stack([uniform_ext_knots(lo, hi, G, 3) for lo, hi in ends])
            coef = rng.normal(size=(4, m, G + 3)).astype(np.float32)
            x = np.tile(specials[:, None], (1, 4))
            _check_layer(LayerSpec(4, m, G, 3, tau, coef, L, SYM_INT8, boundary, oob, per_input=True), x, lk.ALGO_AUTO,
                         what=f"zero-ended domains, per input, b{boundary} o{oob}")
            for row, (lo, hi) in enumerate(ends):                       # the same domains as shared vectors
                _check_layer(LayerSpec(1, m, G, 3, tau[row], coef[row:row + 1], L, SYM_INT8, boundary, oob), x[:, :1].copy(),
                             lk.ALGO_AUTO, what=f"domain [{lo},{hi}] shared b{boundary} o{oob}")


def test_empty_batch_and_argument_errors():
    w = cfg1(B=8)
    s = w.layers[0]
    art, _ = _compile_both(s)
    layer = _device_layer(art, s)
    x0 = torch.empty((0, s.d), dtype=torch.float32, device=DEV)
    y0 = lk.lutkan_forward(layer, x0)
    assert y0.shape == (0, s.m)
    x = torch.from_numpy(w.x).to(DEV)
    with pytest.raises(lk.LutKanError, match="workspace"):
        lk.lutkan_forward(layer, x, workspace=torch.empty(256, dtype=torch.uint8, device=DEV))
    bad = layer.with_contract(7, CLIP_X)
    with pytest.raises(lk.LutKanError, match="boundary"):
        lk.lutkan_forward(bad, x)
    nul = layer.with_contract(CLOSED, CLIP_X)
    nul.c.table = None
    with pytest.raises(lk.LutKanError, match="table"):
        lk.lutkan_forward(nul, x)
    buf = torch.empty((1 << 18,), dtype=torch.float32, device=DEV)
    rc = lk.load_library().lutkan_forward(layer.c, buf.data_ptr(), 8, buf.data_ptr(), None, buf.data_ptr(), buf.numel() * 4, None)
    assert rc == -1 and "alias" in lk.lutkan_last_error()
    torch.cuda.synchronize()


def test_repeatable_bitwise():
    w = random_layer(401, 50, 256, 8, 64, SYM_INT8, CLOSED, CLIP_X, 3000)
    s = w.layers[0]
    art, _ = _compile_both(s)
    xg = torch.from_numpy(w.x).to(DEV)
    for algo in (lk.ALGO_GATHER, lk.ALGO_TILED):
        layer = _device_layer(art, s, algo)
        a = lk.lutkan_forward(layer, xg).clone()
        b = lk.lutkan_forward(layer, xg)
        assert torch.equal(a, b)


def _chain_check(w, what):
    """Each layer against the oracle on the SAME input (the GPU's own activation of the previous layer), and the
    chained entry point bit-identical to the layer-by-layer GPU calls."""
    arts, layers = [], []
    for s in w.layers:
        art, ora = _compile_both(s)
        arts.append((art, ora))
        layers.append(_device_layer(art, s))
    xg = torch.from_numpy(w.x).to(DEV)
    stats = torch.zeros((len(layers), 2), dtype=torch.int64, device=DEV)
    y_model = lk.lutkan_model_forward(layers, xg, stats=stats)
    cur = xg
    for li, (s, (art, ora), layer) in enumerate(zip(w.layers, arts, layers)):
        _say(f"case {what} layer {li}: {s.d}->{s.m} B={cur.shape[0]}")
        nxt = lk.lutkan_forward(layer, cur)
        x_host = cur.cpu().numpy()
        ref = oracle.lut_forward(ora, s.boundary, s.oob, x_host)
        _assert_close(nxt.cpu().numpy(), ref, f"{what} layer {li}")
        st = stats[li].cpu().numpy()
        assert (int(st[0]), int(st[1])) == (ref.oob_count, ref.oob_any_rows)
        cur = nxt
    assert torch.equal(cur, y_model)


def test_cfg2_tabular_two_layer_chain_full_size():
    _chain_check(cfg2(), "cfg2")


@pytest.mark.parametrize("B", [1, 300, 5000])
def test_cfg2_tabular_chain_at_small_batches(B):
    """Up to about 10000 rows every layer of this network runs as a launch of the chain kernel, and lutkan_model_forward
    runs the whole network as one launch of it: same arithmetic, so still bit-identical to the layer-by-layer calls."""
    _chain_check(cfg2(B=B), f"cfg2 B={B}")


@pytest.mark.parametrize("boundary,oob", [(HALF_OPEN, CLIP_X), (HALF_OPEN, ZERO_SPLINE), (CLOSED, CLIP_X), (CLOSED, ZERO_SPLINE)])
def test_cfg5_deep_chain_robustness_matrix(boundary, oob):
    _chain_check(cfg5(B=16384 + 77, boundary=boundary, oob=oob), f"cfg5 b{boundary} o{oob}")


@pytest.mark.parametrize("L", [16, 32, 64, 128])
@pytest.mark.parametrize("scheme", [SYM_INT8, ASYM_UINT8])
def test_cfg3_sweep_point_reduced_batch(L, scheme):
    w = cfg3(L=L, scheme=scheme, B=1024 + 19)
    _check_layer(w.layers[0], w.x, lk.ALGO_AUTO, what=w.name)


@pytest.mark.parametrize("L", [16, 32, 64, 128])
@pytest.mark.parametrize("scheme", [SYM_INT8, ASYM_UINT8])
def test_cfg3_sweep_point_full_batch_every_row(L, scheme):
    """Every point of the L x scheme sweep at its stated batch (16384 rows, the launch plan a user gets): k, l0, In(x),
    w and the counters bit-exact and every output within the tolerance, on all rows."""
    w = cfg3(L=L, scheme=scheme)
    assert w.x.shape[0] == 16384
    _check_layer(w.layers[0], w.x, lk.ALGO_AUTO, what=w.name)


def _sampled_rows_check(w, n_rows, what, seed=0):
    """Full-size launch (the configuration the benchmark times).  The oracle recomputes a seeded random sample of at
    least n_rows rows (plus the first and the last one): k, l0, In(x), w bit-exact and the outputs of both the traced
    and the plain launch within the tolerance on them; the OOB counters are exact over ALL rows."""
    s = w.layers[0]
    art, ora = _compile_both(s)
    layer = _device_layer(art, s)
    xg = torch.from_numpy(w.x).to(DEV)
    B = w.x.shape[0]
    rng = np.random.Generator(np.random.PCG64(seed))
    rows = np.unique(np.concatenate([rng.choice(B, size=min(B, n_rows), replace=False), [0, B - 1]]))
    _say(f"case {what} full size B={B} sampled rows={rows.size}")
    stats = torch.zeros(2, dtype=torch.int64, device=DEV)
    y = lk.lutkan_forward(layer, xg, stats=stats)
    plan = lk.lutkan_last_plan()
    y_t, k, l0, inside, wgt, _ = lk.lutkan_forward_trace(layer, xg)
    assert lk.lutkan_last_plan() == plan.replace("oob; ", "")           # the traced launch is the plain launch's plan
    torch.cuda.synchronize()
    rows_t = torch.from_numpy(rows).to(DEV)
    ref = oracle.lut_forward(ora, s.boundary, s.oob, w.x[rows], trace=True)
    np.testing.assert_array_equal(k[rows_t].cpu().numpy(), ref.k)
    np.testing.assert_array_equal(l0[rows_t].cpu().numpy(), ref.l0)
    np.testing.assert_array_equal(inside[rows_t].cpu().numpy(), ref.inside)
    np.testing.assert_array_equal(wgt[rows_t].cpu().numpy().view(np.uint32), ref.w.view(np.uint32))
    _assert_close(y[rows_t].cpu().numpy(), ref, what)
    _assert_close(y_t[rows_t].cpu().numpy(), ref, what + " (traced launch)")
    T = ora.knots
    inside_all = (w.x >= T[0]) & (w.x <= T[-1]) if s.boundary == CLOSED else (w.x >= T[0]) & (w.x < T[-1])
    st = stats.cpu().numpy()
    assert int(st[0]) == int((~inside_all).sum()) and int(st[1]) == int((~inside_all).any(axis=1).sum())


@pytest.mark.parametrize("boundary,oob", [(HALF_OPEN, CLIP_X), (HALF_OPEN, ZERO_SPLINE), (CLOSED, CLIP_X), (CLOSED, ZERO_SPLINE)])
def test_cfg5_full_batch_chain_every_row(boundary, oob):
    """cfg5 at its full batch (131072 rows, the launch shapes a user gets) under each of the four boundary x policy
    contracts: every layer against the oracle on ALL rows, fed with the GPU's own activations of the previous layer;
    the per-layer OOB counters exact; the chained entry point bit-identical to the layer-by-layer calls."""
    w = cfg5(boundary=boundary, oob=oob)
    B = w.x.shape[0]
    assert B == 131072
    layers, oras = [], []
    for s in w.layers:
        art, ora = _compile_both(s)
        layers.append(_device_layer(art, s))
        oras.append(ora)
    cur = torch.from_numpy(w.x).to(DEV)
    stats = torch.zeros((len(layers), 2), dtype=torch.int64, device=DEV)
    y_model = lk.lutkan_model_forward(layers, cur, stats=stats)
    for li, (s, layer, ora) in enumerate(zip(w.layers, layers, oras)):
        _say(f"case cfg5 b{boundary} o{oob} full batch layer {li}: {s.d}->{s.m} B={B}")
        nxt = lk.lutkan_forward(layer, cur)
        ref = oracle.lut_forward(ora, s.boundary, s.oob, cur.cpu().numpy())
        _assert_close(nxt.cpu().numpy(), ref, f"cfg5 full layer {li}")
        st = stats[li].cpu().numpy()
        assert (int(st[0]), int(st[1])) == (ref.oob_count, ref.oob_any_rows)
        cur = nxt
    assert torch.equal(cur, y_model)


@pytest.mark.parametrize("B", [1, 7, 64, 100, 256, 4096])
def test_cfg4_wide_layer_every_row(B):
    """The widest workload at its batches of 256 and 4096 rows, and at batches of a few rows, where AUTO runs the
    gather kernel with the inputs split into chunks (partial sums added in chunk order): all rows against the oracle."""
    w = cfg4(B=B)
    _check_layer(w.layers[0], w.x, lk.ALGO_AUTO, what=f"cfg4 B={B}")


@pytest.mark.parametrize("L,scheme,B", [(32, ASYM_UINT8, 200), (48, SYM_INT8, 300)], ids=["L32_uint8_200rows", "L48_int8_300rows"])
def test_table_streaming_from_hbm_runs_with_two_slices_in_flight(L, scheme, B):
    """A table of more than 128 MiB at a few hundred rows: the launch waits for the table to stream from HBM and the
    tiled kernel keeps two slices in flight, waiting on a count of its own outstanding copies.  Other slice sizes than
    the widest workload's (two resp. three copies per wave and input at least), both schemes, every row against the oracle."""
    w = random_layer(810 + L, 1024, 1024, 10, L, scheme, CLOSED, ZERO_SPLINE, B, oob_frac=0.1)
    art, _ = _compile_both(w.layers[0])
    assert art.info.table_bytes > 128 << 20
    _check_layer(w.layers[0], w.x, lk.ALGO_TILED, what=w.name)
    layer = _device_layer(art, w.layers[0], lk.ALGO_TILED)
    lk.lutkan_forward(layer, torch.from_numpy(w.x).to(DEV))
    assert " pipe=4; " in lk.lutkan_last_plan(), lk.lutkan_last_plan()


def test_cfg4_wide_layer_largest_batch_sampled_rows():
    """The configuration the benchmark times (1024 -> 1024 at 32768 rows): 4096 random rows against the oracle, the
    OOB counters exact over all rows."""
    _sampled_rows_check(cfg4(B=32768), 4096, "cfg4 B=32768")


@pytest.mark.parametrize("B", [1, 5, 16, 17])
def test_bspline_wide_layer_small_batches(B):
    """The B-spline layer at a few rows: up to 16 rows AUTO takes the gather kernel with the inputs split into chunks."""
    w = cfg4(B=B)
    s = w.layers[0]
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob)
    y = lk.bspline_kan_forward(art.bspline_to_device(DEV), torch.from_numpy(w.x).to(DEV))
    ref = oracle.bspline_forward(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.boundary, s.oob, w.x)
    _assert_close(y.cpu().numpy(), ref, f"bspline cfg4 B={B}")


def test_two_million_rows_sampled():
    """A batch far beyond the workloads (2^21 rows, 2048 row tiles, 1 GiB of lookup records): 64-bit row indexing in
    every kernel, checked on sampled rows and through the exact OOB counters."""
    w = random_layer(351, 64, 48, 6, 32, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 1 << 21)
    _sampled_rows_check(w, 4096, "2^21 rows, 64 -> 48")


# ---------------------------------------------------------------- B-spline baseline
def _check_bspline(s, x, algo, what):
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob,
                            edge_scales=s.edge_scales)
    layer = art.bspline_to_device(DEV, algo)
    _say(f"case bspline {what} d={s.d} m={s.m} G={s.G} boundary={s.boundary} oob={s.oob} B={x.shape[0]} algo={algo}")
    y = lk.bspline_kan_forward(layer, torch.from_numpy(x).to(DEV))
    torch.cuda.synchronize()
    ref = oracle.bspline_forward(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.boundary, s.oob, x, edge_scalars=s.edge_scales)
    _assert_close(y.cpu().numpy(), ref, "bspline " + what)


@pytest.mark.parametrize("case", PROPERTY_CASES[1:] + [(c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7], c[8], c[0] % 2 == 0) for c in TILED_CASES[:5]],
                         ids=lambda c: f"seed{c[0]}")
def test_bspline_layers(case):
    seed, d, m, G, L, scheme, boundary, oob, B, uniform = case
    w = random_layer(seed, d, m, G, L, scheme, boundary, oob, B, uniform=uniform)
    _check_bspline(w.layers[0], w.x, lk.ALGO_GATHER, w.name)
    _check_bspline(w.layers[0], w.x, lk.ALGO_TILED, w.name)


def test_bspline_special_inputs():
    w = random_layer(302, 6, 140, 5, 32, ASYM_UINT8, CLOSED, ZERO_SPLINE, 40)
    x = w.x.copy()
    x[3, 2] = np.nan
    x[5, :] = np.inf
    x[6, :] = -np.inf
    s = w.layers[0]
    for boundary in (HALF_OPEN, CLOSED):
        for oob in (CLIP_X, ZERO_SPLINE):
            s.boundary, s.oob = boundary, oob
            _check_bspline(s, x, lk.ALGO_TILED, "special")
            _check_bspline(s, x, lk.ALGO_GATHER, "special")


def test_bspline_cfg4_every_row():
    w = cfg4(B=4096)
    s = w.layers[0]
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob)
    layer = art.bspline_to_device(DEV)
    y = lk.bspline_kan_forward(layer, torch.from_numpy(w.x).to(DEV))
    ref = oracle.bspline_forward(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.boundary, s.oob, w.x)
    _assert_close(y.cpu().numpy(), ref, "bspline cfg4, all 4096 rows")


# ---------------------------------------------------------------- value_repr = spline_component (Eq. 2, Sec. 4.3 B)
SC_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B
    (501, 1, 1, 4, 16, SYM_INT8, CLOSED, CLIP_X, 50),
    (502, 10, 8, 8, 64, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 1024),
    (503, 7, 3, 5, 32, ASYM_UINT8, CLOSED, ZERO_SPLINE, 333),
    (504, 40, 70, 6, 16, ASYM_UINT8, HALF_OPEN, CLIP_X, 2100),
    (505, 64, 256, 8, 64, SYM_INT8, CLOSED, ZERO_SPLINE, 5000),
    (506, 33, 130, 10, 64, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 1025),
]


@pytest.mark.parametrize("case", SC_CASES, ids=lambda c: f"seed{c[0]}")
def test_spline_component_layers(case):
    seed, d, m, G, L, scheme, boundary, oob, B = case
    w = random_layer(seed, d, m, G, L, scheme, boundary, oob, B, uniform=(seed % 2 == 0), oob_frac=0.5, with_base=True)
    s = w.layers[0]
    _check_layer(s, w.x, lk.ALGO_GATHER, codes=(B * d * m <= 2_000_000), what=w.name)
    _check_layer(s, w.x, lk.ALGO_TILED, what=w.name)
    _check_bspline(s, w.x, lk.ALGO_GATHER, w.name)
    _check_bspline(s, w.x, lk.ALGO_TILED, w.name)


BASE_PRODUCT_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B, per_input, param_fp16      batch * d * m >= 5e8, d a multiple of 32, m >= 64
    (551, 64, 256, 8, 64, SYM_INT8, CLOSED, ZERO_SPLINE, 32768 + 5, False, False),      # ragged last row tile of the product
    (552, 96, 130, 6, 16, ASYM_UINT8, HALF_OPEN, CLIP_X, 41000, False, False),          # ragged column tile (130 of 256 columns)
    (553, 32, 64, 5, 32, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 250001, False, True),        # the narrowest product; float16 parameters
    (554, 128, 128, 5, 32, ASYM_UINT8, CLOSED, CLIP_X, 33000, True, False),             # one knot vector per input
    (555, 1024, 1024, 10, 64, SYM_INT8, CLOSED, CLIP_X, 2048, False, False),            # the widest layer: inputs split, summing pass adds to y
]


@pytest.mark.parametrize("case", BASE_PRODUCT_CASES, ids=lambda c: f"seed{c[0]}")
def test_spline_component_with_the_base_branch_as_a_matrix_product(case):
    """From about 5e8 edge evaluations per call a spline_component layer evaluates its base branch (Eq. 2: s_out * s_base *
    SiLU(x), summed over the inputs) as one [B, d] x [d, m] product on the matrix cores, fp32 operands as three bf16
    pieces, and the LUT edge kernel adds the spline branch on top.  Same bar as every other path: k, l0, In, w bit-exact,
    outputs within the tolerance, on all rows; a NaN input poisons its own row only."""
    seed, d, m, G, L, scheme, boundary, oob, B, per_input, half = case
    if per_input:
        w = per_input_layer(seed, d, m, G, L, scheme, boundary, oob, B, with_base=True)
    else:
        w = random_layer(seed, d, m, G, L, scheme, boundary, oob, B, uniform=(seed % 2 == 0), oob_frac=0.3, with_base=True)
    s = w.layers[0]
    x = w.x.copy()
    x[B // 2, d // 3] = np.nan
    x[B // 3, :] = 30.0                                 # SiLU(x) ~ x
    x[B // 5, :] = -90.0                                # SiLU(x) underflows to -0
    _check_layer(s, x, lk.ALGO_AUTO, what=w.name, param_fp16=half)
    assert "base_product; tiled" in lk.lutkan_last_plan(), lk.lutkan_last_plan()
    # the same layer through the entry points that take the two phases apart, and through the built-in scratch
    art, ora = _compile_both(s, half)
    layer = _device_layer(art, s)
    xg = torch.from_numpy(x).to(DEV)
    y_ref = lk.lutkan_forward(layer, xg)
    ws = torch.empty(lk.lutkan_forward_workspace_bytes(layer, B), dtype=torch.uint8, device=DEV)
    lk.lutkan_forward_locate(layer, xg, ws)
    y_two = lk.lutkan_forward_edges(layer, B, torch.full((B, m), 3.0, dtype=torch.float32, device=DEV), ws)
    same = lambda p, q: bool(((p == q) | (torch.isnan(p) & torch.isnan(q))).all())
    assert same(y_two, y_ref)
    if lk.lutkan_forward_workspace_bytes(layer, B) <= lk.STATIC_SCRATCH_BYTES:
        y_static = lk.lutkan_forward_static_scratch(layer, xg, torch.full((B, m), -3.0, dtype=torch.float32, device=DEV))
        assert same(y_static, y_ref)


@pytest.mark.parametrize("boundary,oob", [(HALF_OPEN, CLIP_X), (HALF_OPEN, ZERO_SPLINE), (CLOSED, CLIP_X), (CLOSED, ZERO_SPLINE)])
def test_case_a_sweep_shape_spline_component(boundary, oob):
    """The paper's controlled-sweep layer (10->8, grid 8, spline_component) with inputs clipped onto the domain."""
    for L, scheme in ((16, ASYM_UINT8), (64, SYM_INT8), (128, ASYM_UINT8)):
        w = case_a(seed=1, L=L, scheme=scheme, boundary=boundary, oob=oob)
        _check_layer(w.layers[0], w.x, lk.ALGO_AUTO, codes=True, what=w.name)


def test_spline_component_special_inputs():
    w = random_layer(507, 6, 140, 5, 32, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 40, with_base=True)
    x = w.x.copy()
    x[3, 2] = np.nan
    x[5, :] = 80.0          # SiLU(x) ~ x, exp(-x) underflows
    x[6, :] = -120.0        # exp(-x) overflows to inf: SiLU -> -0
    x[7, :] = np.inf
    s = w.layers[0]
    for algo in (lk.ALGO_GATHER, lk.ALGO_TILED):
        _check_layer(s, x[:7], algo, what="sc special")


STATS_CASES = [
    # seed, B, d, m, boundary, spread of x around the domain [-1, 1]
    (701, 1, 1, 1, CLOSED, 1.5),
    (702, 63, 7, 5, HALF_OPEN, 1.2),
    (703, 1000, 70, 130, CLOSED, 1.05),
    (704, 4099, 64, 8, HALF_OPEN, 1.0),          # U(-1, 1): every row in-range
    (705, 300, 300, 3, CLOSED, 3.0),             # every row has an input outside
    (706, 20000, 16, 64, HALF_OPEN, 1.01),
]


@pytest.mark.parametrize("case", STATS_CASES, ids=lambda c: f"seed{c[0]}")
def test_error_stats_kernel(case):
    """Sec. 5.6 statistics reduced on the device against their plain definition: counts and maxima exact, fp64 sums
    up to the order of summation."""
    seed, B, d, m, boundary, spread = case
    rng = np.random.Generator(np.random.PCG64(seed))
    x = rng.uniform(-spread, spread, size=(B, d)).astype(np.float32)
    x.reshape(-1)[rng.integers(0, B * d, size=max(1, B * d // 50))] = np.float32(1.0)      # inputs exactly on t_K
    y = rng.normal(size=(B, m)).astype(np.float32)
    r = (y + rng.normal(scale=1e-3, size=(B, m))).astype(np.float32)
    if B > 10:
        x[B // 2, 0] = np.nan
        y[B // 3, m // 2] = np.nan
    _say(f"case stats seed={seed} B={B} d={d} m={m} boundary={boundary}")
    got = lk.lutkan_error_stats(torch.from_numpy(y).to(DEV), torch.from_numpy(r).to(DEV), torch.from_numpy(x).to(DEV),
                                -1.0, 1.0, boundary)
    want = oracle.error_stats(y, r, x, -1.0, 1.0, boundary)
    _same_error_summary(got, want)


def _same_error_summary(got, want):
    """Every field of lutkan_error_summary against the oracle's: counts, maxima and the OOB fraction exact, the fp64
    sums and means up to the order of summation."""
    assert set(got) == set(want)
    for key in ("rows_in", "rows_oob", "nan_in", "nan_oob", "max_abs_in", "max_abs_oob", "oob_any_frac"):
        assert got[key] == want[key], key
    for key in ("sum_abs_in", "sum_abs_oob", "mae_in", "mae_oob"):
        if np.isnan(want[key]):
            assert np.isnan(got[key]), key
        else:
            assert abs(got[key] - want[key]) <= 1e-12 * abs(want[key]) + 1e-300, key


def test_error_stats_mean_leaves_nan_outputs_out_of_the_count():
    """NaN outputs inside both subsets (several per subset, so that rows * m and the number of differences that exist
    differ visibly): the device divides each sum by the latter, as the oracle does; a subset of NaN outputs only has
    no mean."""
    rng = np.random.Generator(np.random.PCG64(720))
    B, d, m = 500, 6, 10
    x = rng.uniform(-1.1, 1.1, size=(B, d)).astype(np.float32)
    y = rng.normal(size=(B, m)).astype(np.float32)
    r = (y + rng.normal(scale=1e-2, size=(B, m))).astype(np.float32)
    y.reshape(-1)[rng.choice(B * m, size=B * m // 5, replace=False)] = np.nan
    _say(f"case stats with NaN outputs in both subsets B={B} d={d} m={m}")
    got = lk.lutkan_error_stats(torch.from_numpy(y).to(DEV), torch.from_numpy(r).to(DEV), torch.from_numpy(x).to(DEV),
                                -1.0, 1.0, CLOSED)
    want = oracle.error_stats(y, r, x, -1.0, 1.0, CLOSED)
    assert want["nan_in"] > 50 and want["nan_oob"] > 50 and want["rows_in"] > 50 and want["rows_oob"] > 50
    _same_error_summary(got, want)
    assert abs(got["mae_in"] - got["sum_abs_in"] / (got["rows_in"] * m - got["nan_in"])) <= 1e-15
    assert got["mae_in"] > 1.1 * got["sum_abs_in"] / (got["rows_in"] * m)          # the other denominator is 20 % larger
    y[:] = np.nan
    got = lk.lutkan_error_stats(torch.from_numpy(y).to(DEV), torch.from_numpy(r).to(DEV), torch.from_numpy(x).to(DEV),
                                -1.0, 1.0, CLOSED)
    _same_error_summary(got, oracle.error_stats(y, r, x, -1.0, 1.0, CLOSED))
    assert np.isnan(got["mae_in"]) and np.isnan(got["mae_oob"]) and got["nan_in"] == got["rows_in"] * m


def test_error_stats_of_a_lut_layer_against_its_spline_layer():
    """The protocol end to end on one layer: LUT output vs B-spline output, subsets by In(x)."""
    w = random_layer(711, 8, 128, 5, 32, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 8192)
    s = w.layers[0]
    art, _ = _compile_both(s)
    xg = torch.from_numpy(w.x).to(DEV)
    y_lut = lk.lutkan_forward(_device_layer(art, s), xg)
    y_ref = lk.bspline_kan_forward(art.bspline_to_device(DEV).with_contract(CLOSED, CLIP_X), xg)
    got = lk.lutkan_error_stats(y_lut, y_ref, xg, float(art.knots[0]), float(art.knots[-1]), s.boundary)
    torch.cuda.synchronize()
    want = oracle.error_stats(y_lut.cpu().numpy(), y_ref.cpu().numpy(), w.x, art.knots[0], art.knots[-1], s.boundary)
    assert (got["rows_in"], got["rows_oob"]) == (want["rows_in"], want["rows_oob"]) and min(got["rows_in"], got["rows_oob"]) > 100
    assert got["max_abs_in"] == want["max_abs_in"] and got["max_abs_oob"] == want["max_abs_oob"]
    assert abs(got["mae_in"] - want["mae_in"]) <= 1e-12 * want["mae_in"]
    assert got["mae_oob"] > 2 * got["mae_in"]                     # zero_spline drops the OOB inputs' contributions


def test_model_forward_replays_correctly_from_a_hip_graph():
    """The chain launches only kernels (no allocation, no memset, no synchronisation), so it can be captured;
    every replay, with eager work in between, reproduces the eager result bit for bit."""
    w = cfg2(B=5000)
    arts = [lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob) for s in w.layers]
    layers = [a.to_device(DEV) for a in arts]
    x = torch.from_numpy(w.x).to(DEV)
    B = x.shape[0]
    ws = torch.empty(lk.lutkan_model_workspace_bytes(layers, B), dtype=torch.uint8, device=DEV)
    y = torch.empty((B, layers[-1].m), dtype=torch.float32, device=DEV)
    stats = torch.zeros((len(layers), 2), dtype=torch.int64, device=DEV)
    _say(f"case graph capture {w.name} B={B}")
    lk.lutkan_model_forward(layers, x, y, stats=stats, workspace=ws)           # warm-up: one-time kernel attributes
    torch.cuda.synchronize()
    y_eager, stats_eager = y.clone(), stats.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        lk.lutkan_model_forward(layers, x, y, stats=stats, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lk.lutkan_model_forward(layers, x, y, stats=stats, workspace=ws)
    for _ in range(3):
        y.fill_(7.0)
        stats.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, y_eager) and torch.equal(stats, stats_eager)
        lk.lutkan_model_forward(layers, x, y, workspace=ws)                    # eager work between replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("B", [256, 5000])
def test_fused_chain_replays_correctly_from_a_hip_graph(B):
    """One kernel launch and nothing else: captured after one eager call (which sets the kernel's one-time
    attribute), every replay with eager work in between reproduces the eager result bit for bit."""
    w = cfg2(B=B)
    arts = [lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob) for s in w.layers]
    layers = [a.to_device(DEV) for a in arts]
    x = torch.from_numpy(w.x).to(DEV)
    y = torch.empty((B, layers[-1].m), dtype=torch.float32, device=DEV)
    stats = torch.zeros((len(layers), 2), dtype=torch.int64, device=DEV)
    _say(f"case graph capture of the fused chain {w.name} B={B}")
    lk.lutkan_chain_forward(layers, x, y, stats=stats)
    torch.cuda.synchronize()
    y_eager, stats_eager = y.clone(), stats.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        lk.lutkan_chain_forward(layers, x, y, stats=stats)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lk.lutkan_chain_forward(layers, x, y, stats=stats)
    for _ in range(3):
        y.fill_(7.0)
        stats.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, y_eager) and torch.equal(stats, stats_eager)
        lk.lutkan_chain_forward(layers, x, y)                                  # eager work between replays
        torch.cuda.synchronize()


def test_random_shapes_and_contracts():
    """Sixty layers with shapes, grids, table sizes and contracts drawn at random (seeded), covering every tile width,
    ragged tiles and batches, both value representations, both parameter dtypes and both kernel families; the LUT
    layer (trace and plain launch, counters) and the B-spline layer against the oracle."""
    rng = np.random.Generator(np.random.PCG64(2024))
    worst = 0.0
    for it in range(60):
        G = int(rng.choice([1, 2, 3, 5, 8, 10, 17, 33, 64]))
        L = int(rng.choice([2, 3, 5, 16, 31, 64, 128, 512]))
        L = min(L, 65535 // G)
        d = int(rng.integers(1, 41))
        m = int(rng.choice([1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 31, 32, 33, 64, 65, 100, 128, 129, 200, 300]))
        B = int(rng.choice([1, 2, 15, 16, 17, 63, 64, 65, 255, 256, 257, 1000, 1024, 1025, 2500]))
        scheme, boundary, oob = (int(rng.integers(0, 2)) for _ in range(3))
        base = bool(rng.integers(0, 2))
        half = bool(rng.integers(0, 2))
        algo = int(rng.choice([lk.ALGO_AUTO, lk.ALGO_GATHER]))
        w = random_layer(2000 + it, d, m, G, L, scheme, boundary, oob, B, uniform=bool(rng.integers(0, 2)), with_base=base)
        s = w.layers[0]
        _say(f"case random {it}: d={d} m={m} G={G} L={L} B={B} scheme={scheme} boundary={boundary} oob={oob} base={base} "
             f"fp16={half} algo={algo}")
        worst = max(worst, _check_layer(s, w.x, algo, what=w.name, param_fp16=half))
        yb = lk.bspline_kan_forward(_compile_both(s, half)[0].bspline_to_device(DEV), torch.from_numpy(w.x).to(DEV))
        torch.cuda.synchronize()
        refb = oracle.bspline_forward(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.boundary, s.oob, w.x, edge_scalars=s.edge_scales)
        worst = max(worst, _assert_close(yb.cpu().numpy(), refb, w.name + " bspline"))
    _say(f"random layers: worst error / tolerance = {worst:.3f}")


# ---- fused chain: the whole narrow network in one launch ----

def _narrow_chain(seed, widths, G, L, scheme, boundary, oob, B, with_base=False, lo=-2.0, hi=2.0):
    """Layers of a narrow network on [lo, hi] with coefficients ~ N(0, 1/sqrt(d)); x ~ N(0,1) with heavy tails."""
    from lutkan_inputs import LayerSpec, draw_edge_scales, uniform_ext_knots
    rng = np.random.Generator(np.random.PCG64(seed))
    layers = []
    for d, m in zip(widths[:-1], widths[1:]):
        coef = rng.normal(0.0, 1.0 / np.sqrt(d), size=(d, m, G + 3)).astype(np.float32)
        s = LayerSpec(d, m, G, 3, uniform_ext_knots(lo, hi, G, 3), coef, L, scheme, boundary, oob)
        if with_base:
            s.edge_scales = draw_edge_scales(rng, d, m)
        layers.append(s)
    x = np.where(rng.random((B, widths[0])) < 0.1, rng.standard_t(3.0, size=(B, widths[0])), rng.normal(size=(B, widths[0]))).astype(np.float32)
    return layers, x


def _fused_chain_check(specs, x, what, param_fp16=False):
    """Every layer of the fused launch against the oracle on the SAME input (the launch's own hidden activation of
    the previous layer), its counters against the oracle's, and the result against the layer-by-layer chain."""
    compiled = [_compile_both_uncached(s, param_fp16) for s in specs]
    layers = [_device_layer(art, s) for s, (art, _) in zip(specs, compiled)]
    B = x.shape[0]
    xg = torch.from_numpy(x).to(DEV)
    hidden = torch.full((B * sum(s.m for s in specs[:-1]) + 1,), float("nan"), dtype=torch.float32, device=DEV)
    stats = torch.zeros((len(specs), 2), dtype=torch.int64, device=DEV)
    _say(f"case {what}: fused chain {[s.d for s in specs] + [specs[-1].m]} B={B} fp16={param_fp16}")
    y = lk.lutkan_chain_forward(layers, xg, stats=stats, hidden=hidden)
    y_plain = lk.lutkan_chain_forward(layers, xg)
    torch.cuda.synchronize()
    assert torch.equal(y, y_plain) or np.array_equal(np.isnan(y.cpu().numpy()), np.isnan(y_plain.cpu().numpy()))
    h = hidden.cpu().numpy()
    assert np.isnan(h[-1])                                # nothing written past the trace
    cur, off, worst = x, 0, 0.0
    for li, (s, (art, ora)) in enumerate(zip(specs, compiled)):
        ref = oracle.lut_forward(ora, s.boundary, s.oob, cur, edge_scalars=s.edge_scales)
        if li + 1 < len(specs):
            nxt = h[off:off + B * s.m].reshape(B, s.m)
            off += B * s.m
        else:
            nxt = y.cpu().numpy()
        worst = max(worst, _assert_close(nxt, ref, f"{what} layer {li}"))
        st = stats[li].cpu().numpy()
        assert (int(st[0]), int(st[1])) == (ref.oob_count, ref.oob_any_rows), f"{what} layer {li} counters"
        cur = nxt
    y_model = lk.lutkan_model_forward(layers, xg).cpu().numpy()
    scale = np.abs(y_model[np.isfinite(y_model)]).max() if np.isfinite(y_model).any() else 1.0
    ok = np.isfinite(y_model)
    assert np.abs(y.cpu().numpy()[ok] - y_model[ok]).max() <= 1e-3 * max(scale, 1.0)
    return worst


def _compile_both_uncached(s, param_fp16):
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob,
                            edge_scales=s.edge_scales, param_dtype=lk.PARAM_FP16 if param_fp16 else lk.PARAM_FP32)
    ora = oracle.compile_layer(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, param_fp16=param_fp16)
    assert np.array_equal(art.q, ora.q) and np.array_equal(art.scale, ora.scale) and np.array_equal(art.y_min, ora.y_min)
    return art, ora


FUSED_CHAIN_CASES = [
    # seed, widths, G, L, scheme, boundary, oob, B, with_base, param_fp16
    (901, (78, 16, 2), 5, 64, ASYM_UINT8, CLOSED, CLIP_X, 256, False, False),          # the tabular shape at the latency batch
    (902, (78, 32, 16, 1), 5, 64, SYM_INT8, CLOSED, CLIP_X, 256, True, False),         # the case study's network (Sec. 8)
    (903, (78, 32, 16, 1), 5, 64, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 1027, True, True),
    (904, (10, 8), 8, 16, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 1, False, False),           # one layer, one row
    (905, (5, 64, 3, 64, 4), 3, 8, ASYM_UINT8, CLOSED, ZERO_SPLINE, 3, False, True),    # 64-column layers, one group per wave
    (906, (1024, 4, 1), 4, 32, SYM_INT8, CLOSED, CLIP_X, 70, False, False),             # the widest input, 16 groups of inputs
    (907, (3, 5, 7, 9, 11, 13, 15, 17, 2), 6, 16, ASYM_UINT8, HALF_OPEN, CLIP_X, 4099, True, False),   # eight layers
]


@pytest.mark.parametrize("case", FUSED_CHAIN_CASES, ids=lambda c: f"seed{c[0]}")
def test_fused_chain(case):
    seed, widths, G, L, scheme, boundary, oob, B, with_base, half = case
    specs, x = _narrow_chain(seed, widths, G, L, scheme, boundary, oob, B, with_base)
    if B > 10:
        x[B // 2, 0] = np.nan                       # poisons its own row only
        x[B // 3, :] = 50.0                         # every input out of domain
    _fused_chain_check(specs, x, f"fused seed{seed}", half)


@pytest.mark.parametrize("B", [3, 300, 3000])
def test_fused_chain_with_one_knot_vector_per_input(B):
    """A network whose layers each have per-input knot vectors (the grids of a model after per-feature grid updates):
    the fused launch locates every input on its own vector, read from global memory."""
    rng = np.random.Generator(np.random.PCG64(930))
    widths, G, L = (20, 9, 5, 2), 6, 32
    specs = []
    for li, (d, m) in enumerate(zip(widths[:-1], widths[1:])):
        s = per_input_layer(931 + li, d, m, G, L, ASYM_UINT8 if li % 2 else SYM_INT8, HALF_OPEN, ZERO_SPLINE, 4, with_base=(li == 1)).layers[0]
        s.coef = (s.coef / np.sqrt(d)).astype(np.float32)
        specs.append(s)
    x = per_input_layer(931, widths[0], widths[1], G, L, SYM_INT8, HALF_OPEN, ZERO_SPLINE, B).x     # covers layer 0's own domains
    compiled = [_compile_both(s) for s in specs]
    layers = [_device_layer(art, s) for s, (art, _) in zip(specs, compiled)]
    xg = torch.from_numpy(x).to(DEV)
    hidden = torch.zeros(B * sum(widths[1:-1]), dtype=torch.float32, device=DEV)
    stats = torch.zeros((len(specs), 2), dtype=torch.int64, device=DEV)
    _say(f"case fused chain with per-input knots {widths} B={B}")
    y = lk.lutkan_chain_forward(layers, xg, stats=stats, hidden=hidden)
    y_model = lk.lutkan_model_forward(layers, xg)
    torch.cuda.synchronize()
    assert torch.equal(y, y_model)                          # every layer is a small one: the same single launch
    h, cur, off = hidden.cpu().numpy(), x, 0
    for li, (s, (art, ora)) in enumerate(zip(specs, compiled)):
        ref = oracle.lut_forward(ora, s.boundary, s.oob, cur, edge_scalars=s.edge_scales)
        nxt = h[off:off + B * s.m].reshape(B, s.m) if li + 1 < len(specs) else y.cpu().numpy()
        off += B * s.m
        _assert_close(nxt, ref, f"per-input chain layer {li}")
        st = stats[li].cpu().numpy()
        assert (int(st[0]), int(st[1])) == (ref.oob_count, ref.oob_any_rows)
        cur = nxt


@pytest.mark.parametrize("boundary", [HALF_OPEN, CLOSED])
def test_every_kernel_locates_bit_exactly_through_a_revealing_table(boundary):
    """A one-edge layer whose table makes the output spell out the lookup: codes q[k][l] = l, alpha_k = 2^k, y_min = 0,
    so y = 2^k * (l0 + w) = 2^k * z exactly (z - l0 = w and l0 + w = z are exact in fp32).  The oracle's (k, l0, w)
    therefore fix the output of every edge kernel bit for bit -- also of the kernels that have no trace outputs
    (the tiled kernel and the fused chain)."""
    G, L, B = 7, 64, 4000
    rng = np.random.Generator(np.random.PCG64(77 + boundary))
    knots = np.unique(np.sort(rng.uniform(-2.0, 3.0, size=G + 1)).astype(np.float32))   # no knot at 0: a subnormal x
    # next to it gives a subnormal z, which the tiled kernel's 2^-24-scaled sums flush (far below the tolerance)
    K = knots.size - 1
    q = np.tile(np.arange(L, dtype=np.uint8), (1, K, 1))
    scale = (2.0 ** np.arange(K)).astype(np.float32).reshape(1, K)
    art = lk.lutkan_artifact_from_arrays(1, 1, knots, q, scale, np.zeros((1, K), np.float32), boundary, CLIP_X)
    x = rng.uniform(knots[0] - 0.5, knots[-1] + 0.5, size=(B, 1)).astype(np.float32)
    special = np.concatenate([knots, np.nextafter(knots, np.float32(-np.inf)), np.nextafter(knots, np.float32(np.inf))])
    x[:special.size, 0] = special
    ora = SimpleNamespace(d=1, m=1, K=K, L=L, scheme=ASYM_UINT8, knots=knots, q=q, scale=scale, y_min=np.zeros((1, K), np.float32))
    ref = oracle.lut_forward(ora, boundary, CLIP_X, x, trace=True)
    z = ref.l0[:, 0].astype(np.float32) + ref.w[:, 0]
    want = np.ldexp(z, ref.k[:, 0]).astype(np.float32)
    xg = torch.from_numpy(x).to(DEV)
    outs = {"tiled": lk.lutkan_forward(art.to_device(DEV, lk.ALGO_TILED), xg),
            "gather": lk.lutkan_forward(art.to_device(DEV, lk.ALGO_GATHER), xg),
            "chain, a work-group per row": lk.lutkan_chain_forward([art.to_device(DEV)], xg[:900].contiguous()),
            "chain, a wave per row": lk.lutkan_chain_forward([art.to_device(DEV)], xg),
            "auto": lk.lutkan_forward(art.to_device(DEV), xg)}
    torch.cuda.synchronize()
    for name, y in outs.items():
        got = y.cpu().numpy()[:, 0]
        np.testing.assert_array_equal(got.view(np.uint32), want[:got.size].view(np.uint32), err_msg=name)


def test_fused_chain_refuses_what_it_cannot_hold():
    specs, x = _narrow_chain(920, (8, 128, 4), 4, 8, SYM_INT8, CLOSED, CLIP_X, 8)
    layers = [_device_layer(_compile_both_uncached(s, False)[0], s) for s in specs]
    xg = torch.from_numpy(x).to(DEV)
    with pytest.raises(lk.LutKanError) as e:        # a 128-column layer
        lk.lutkan_chain_forward(layers, xg)
    assert str(e.value).startswith("[-5]")
    with pytest.raises(lk.LutKanError) as e:        # widths that do not chain
        lk.lutkan_chain_forward([layers[0], layers[0]], xg)
    assert str(e.value).startswith("[-2]")


def test_last_plan_reports_what_auto_dispatch_launched():
    """lutkan_last_plan names the kernels of the last forward call: the dispatch rules of algo = AUTO, observed."""
    w = cfg4(B=4096)
    s = w.layers[0]
    art, _ = _compile_both(s)
    layer = _device_layer(art, s)
    xg = torch.from_numpy(w.x).to(DEV)
    _say("case last plan: cfg4 at 1, 64 and 4096 rows")
    import re

    def tiled_groups(plan, B, jt, n_tiles):
        """Work-groups of the tiled launch named in `plan`, and its chunk count: the launch shape comes out of a
        fitted cost model, so only its invariants are asserted -- a legal row-step count, whole rounds' worth of
        work-groups, and a summing pass exactly when the inputs were split."""
        mt = re.search(r"tiled np=(\d+) split=(\d+) pipe=(\d); ", plan)
        assert mt, plan
        np_, split, pipe = int(mt.group(1)), int(mt.group(2)), int(mt.group(3))
        rows_per_wave = (64 // (jt // 4)) * np_
        assert np_ in (1, 2, 4, 8, 16) and rows_per_wave <= 64 and 1 <= split <= 128 and pipe in (2, 3, 4)
        assert plan.endswith("sum; ") == (split > 1), plan
        return -(-B // (16 * rows_per_wave)) * n_tiles * split, split

    lk.lutkan_forward(layer, xg[:1])
    plan = lk.lutkan_last_plan()                                                # a few rows: only the touched table rows,
    assert re.fullmatch(r"locate; gather split=(\d+); sum; ", plan), plan      # the inputs split over the GPU
    lk.lutkan_forward(layer, xg[:64])
    assert lk.lutkan_last_plan().startswith("locate; gather split=")
    lk.lutkan_forward(layer, xg)
    plan = lk.lutkan_last_plan()
    assert plan.startswith("locate; tiled np="), plan
    groups, _ = tiled_groups(plan, 4096, art.info.jt, art.info.n_tiles)
    assert groups >= 256, plan                                                  # at least one work-group per compute unit
    assert " pipe=3; " in plan, plan                                            # three slice buffers fit: reads carried across inputs
    lk.lutkan_forward(layer, xg[:256])                                          # the 686 MiB table streaming from HBM is the launch's time:
    assert re.search(r"tiled np=\d+ split=\d+ pipe=4; ", lk.lutkan_last_plan()), lk.lutkan_last_plan()      # two slices in flight
    lk.lutkan_forward(layer, xg)
    stats = torch.zeros(2, dtype=torch.int64, device=DEV)
    lk.lutkan_forward(layer, xg, stats=stats)
    assert lk.lutkan_last_plan() == plan.replace("locate; ", "locate; oob; ")   # the counters add one launch, nothing else
    lk.bspline_kan_forward(art.bspline_to_device(DEV), xg)
    assert re.fullmatch(r"bspline_matrix np=1 split=\d+ slots=16; (sum; )?", lk.lutkan_last_plan()), lk.lutkan_last_plan()
    _say("case last plan: cfg2 at 300, 5000, 20000 and 40000 rows")
    w2 = cfg2(B=40000)
    layers = []
    keep = []
    for s2 in w2.layers:
        a2, _ = _compile_both(s2)
        keep.append(a2)
        layers.append(_device_layer(a2, s2))
    x2 = torch.from_numpy(w2.x).to(DEV)
    lk.lutkan_model_forward(layers, x2[:300])
    assert lk.lutkan_last_plan() == "chain layers=2 wpr=4; "                   # every layer small: one launch, a work-group per row
    lk.lutkan_model_forward(layers, x2[:5000])
    assert lk.lutkan_last_plan() == "chain layers=2 wpr=1; "                   # beyond 1024 rows: a wave per row
    lk.lutkan_forward(layers[0], x2[:300])
    assert lk.lutkan_last_plan() == "chain layers=1 wpr=4; "                   # a single small layer runs as a one-layer chain
    lk.lutkan_model_forward(layers, x2[:20000])
    plan = lk.lutkan_last_plan()                                               # 78x16 has outgrown the chain kernel, 16x2 has not yet
    assert re.fullmatch(r"narrow split=\d+ waves=\d+; (sum; )?chain layers=1 wpr=1; ", plan), plan
    lk.lutkan_model_forward(layers, x2)
    plan = lk.lutkan_last_plan()
    assert re.fullmatch(r"(narrow split=\d+ waves=\d+; (sum; )?){2}", plan), plan     # large batches: the narrow kernel per layer
    torch.cuda.synchronize()


def test_measurement_probes_report_their_work():
    """The peak-rate probes behind the roofline terms: each kind launches and reports the work of one launch (the
    count the rate is computed from), which follows from the launch shape and the iteration count; the rate itself is
    only required to be a finite positive number here -- its value belongs to the benchmark's record, not to a test."""
    buf = torch.zeros((1 << 30) // 4 + 4, dtype=torch.float32, device=DEV)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    kinds = {lk.PROBE_VALU_FMA: 2048, lk.PROBE_VALU_FMAC: 2048, lk.PROBE_VALU_MIX: 2048, lk.PROBE_LDS_READ: 512, lk.PROBE_L2_READ: 4,
             lk.PROBE_HBM_READ: 2}
    for kind, iters in kinds.items():
        lk.lutkan_probe_launch(kind, buf, iters)             # warm-up
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        work = lk.lutkan_probe_launch(kind, buf, iters)
        e1.record()
        torch.cuda.synchronize()
        half = lk.lutkan_probe_launch(kind, buf, iters // 2)
        torch.cuda.synchronize()
        rate = work / (e0.elapsed_time(e1) * 1e-3)
        _say(f"probe kind {kind}: work {work:.4g}, {rate:.3g} per second on {cus} compute units")
        assert work > 0 and work == 2 * half                 # proportional to the iterations inside the kernel
        assert np.isfinite(rate) and rate > 0
    assert lk.lutkan_probe_launch(lk.PROBE_HBM_READ, buf, 2) == 2.0 * (buf.numel() * 4 - 16)      # the buffer, once per pass
    with pytest.raises(lk.LutKanError):
        lk.lutkan_probe_launch(99, buf, 1)
    with pytest.raises(lk.LutKanError):
        lk.lutkan_probe_launch(lk.PROBE_HBM_READ, buf[:1024], 1)


# ---------------------------------------------------------------- the B-spline layer on the matrix cores
MATRIX_CASES = [
    # seed, d, m, G, boundary, oob, B, uniform: 8 slots to G = 5, 12 to 9, 16 to 13; 32, 64 and 128 columns per work-group
    (901, 1, 1, 1, CLOSED, CLIP_X, 1, True),
    (902, 3, 5, 5, HALF_OPEN, ZERO_SPLINE, 33, False),
    (903, 8, 32, 5, CLOSED, ZERO_SPLINE, 256, True),          # exactly one stage, one work-group of rows
    (904, 9, 33, 4, HALF_OPEN, CLIP_X, 257, False),           # one input and one row over
    (905, 20, 64, 6, CLOSED, CLIP_X, 513, False),             # the smallest layer of 12 slots; rows of whole 16-byte vectors
    (906, 21, 65, 13, HALF_OPEN, ZERO_SPLINE, 511, True),     # the largest; odd rows
    (907, 132, 129, 5, CLOSED, ZERO_SPLINE, 1000, False),     # inputs split, two column tiles, a chunk that ends inside a stage
    (908, 130, 300, 10, HALF_OPEN, ZERO_SPLINE, 700, False),
    (909, 64, 8, 5, CLOSED, CLIP_X, 140000, True),            # two row tiles per wave on narrow columns
    (910, 68, 64, 12, HALF_OPEN, CLIP_X, 70001, False),
    (911, 512, 400, 7, CLOSED, ZERO_SPLINE, 5003, False),     # four column tiles, 1e9 edges
]


@pytest.mark.parametrize("case", MATRIX_CASES, ids=lambda c: f"seed{c[0]}")
def test_bspline_layer_on_the_matrix_cores(case):
    """Against the oracle at the edges of the kernel's tiles, with NaN and infinite inputs in one row each."""
    seed, d, m, G, boundary, oob, B, uniform = case
    w = random_layer(seed, d, m, G, 2, SYM_INT8, boundary, oob, B, uniform=uniform)
    s, x = w.layers[0], w.x
    if B > 20:
        x[3, d // 2] = np.nan
        x[5, :] = np.inf
        x[B - 1, 0] = -np.inf
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob)
    layer = art.bspline_to_device(DEV)
    _say(f"case bspline matrix d={d} m={m} G={G} boundary={boundary} oob={oob} B={B}")
    xg = torch.from_numpy(x).to(DEV)
    y = lk.bspline_kan_forward(layer, xg)
    plan = lk.lutkan_last_plan()
    assert f"slots={8 if G <= 5 else 12 if G <= 9 else 16}; " in plan and plan.startswith("bspline_matrix "), plan
    shifted = torch.empty(B * d + 1, dtype=torch.float32, device=DEV)[1:].view(B, d).copy_(xg)      # rows off the 16-byte grid
    y_shifted = lk.bspline_kan_forward(layer, shifted)
    torch.cuda.synchronize()
    ref = oracle.bspline_forward(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.boundary, s.oob, x)
    _assert_close(y.cpu().numpy(), ref, f"bspline matrix {w.name}")
    assert np.array_equal(y.cpu().numpy(), y_shifted.cpu().numpy(), equal_nan=True)


CHUNK_CASES = [
    # seed, d, m, G, L, scheme, B, row steps, chunks: column tiles (3, 10, 11, 15) that do not divide 256
    (641, 1000, 180, 8, 64, ASYM_UINT8, 5000, 16, 17),     # 255 work-groups; without the search inside a round 8 chunks of half row tiles
    (642, 1024, 700, 10, 64, SYM_INT8, 1000, 16, 23),      # 253; without it 24 chunks = 264
    (643, 900, 900, 8, 64, ASYM_UINT8, 600, 16, 17),       # 255; without it 8 chunks of half row tiles
    (644, 577, 623, 9, 80, SYM_INT8, 544, 16, 49),         # 25 chunks end inside the round, but their sums are twice as long
    (645, 141, 161, 8, 64, ASYM_UINT8, 3867, 8, 8),        # 10 chunks are priced 7 % lower, less than an eighth
    (646, 512, 600, 5, 32, SYM_INT8, 1500, 8, 8),          # 12 chunks on the fp32 values, a table beyond the caches: left out
]


@pytest.mark.parametrize("case", CHUNK_CASES, ids=lambda c: f"seed{c[0]}")
def test_chunks_of_column_tiles_that_do_not_divide_the_chip(case):
    """A chunk count that ends inside a round of 256 work-groups is taken where the rule allows it, and only there."""
    seed, d, m, G, L, scheme, B, np_, split = case
    w = random_layer(seed, d, m, G, L, scheme, CLOSED, CLIP_X, B)
    s = w.layers[0]
    art, ora = _compile_both(s)
    layer = _device_layer(art, s)
    _say(f"case chunks d={d} m={m} B={B}")
    y = lk.lutkan_forward(layer, torch.from_numpy(w.x).to(DEV))
    assert f"tiled np={np_} split={split} " in lk.lutkan_last_plan(), lk.lutkan_last_plan()
    _assert_close(y.cpu().numpy(), oracle.lut_forward(ora, s.boundary, s.oob, w.x), f"chunks {w.name}")


# widths, rows, L, scheme, with stats, what runs: without a workspace (0) or with one (1)
WITHOUT_WORKSPACE = [((10, 8), 1024, 64, SYM_INT8, False, 0), ((78, 16, 2), 256, 64, ASYM_UINT8, True, 0), ((78, 16, 2), 0, 64, ASYM_UINT8, False, 0),
                     ((256, 256), 16, 64, SYM_INT8, True, 0), ((256, 256), 4000, 64, SYM_INT8, False, 1), ((78, 16), 65536, 64, ASYM_UINT8, True, 0),
                     ((1000, 30), 9000, 16, SYM_INT8, False, 1), ((40, 60, 60, 10), 5000, 32, ASYM_UINT8, True, 1), ((200, 300), 1000, 48, ASYM_UINT8, True, 1)]


@pytest.mark.parametrize("case", WITHOUT_WORKSPACE, ids=lambda c: "-".join(map(str, c[0])) + f"x{c[1]}")
def test_forward_without_a_workspace(case):
    """A call without a workspace either is the call with one, bit for bit on the same route, or launches nothing and says how
    much it needs; the binding returns the same outputs and counters both ways."""
    import ctypes as C
    widths, B, L, scheme, with_stats, needs = case
    layers, w = [], None
    for n, (d, m) in enumerate(zip(widths[:-1], widths[1:])):
        w = random_layer(640 + n, d, m, 5, L, scheme, CLOSED, CLIP_X, max(B, 1))
        s = w.layers[0]
        layers.append(lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob).to_device(DEV))
        x = w.x if n == 0 else x
    xg = torch.from_numpy(x[:B].copy()).to(DEV)
    n, lib, need = len(layers), lk.load_library(), C.c_size_t(77)
    arr = (type(layers[0].c) * n)(*[l.c for l in layers])
    stats = [torch.zeros((n, 2), dtype=torch.int64, device=DEV) if with_stats else None for _ in range(3)]
    ptr = [t.data_ptr() if t is not None else None for t in stats]
    room = lk.lutkan_model_workspace_bytes(layers, B) if n > 1 else lk.lutkan_forward_workspace_bytes(layers[0], B)
    ws = torch.empty(max(room, 256), dtype=torch.uint8, device=DEV)
    y0, y1 = (torch.full((B, widths[-1]), -7.0, device=DEV) for _ in range(2))
    _say(f"case without a workspace {widths} B={B}")
    stream = torch.cuda.current_stream().cuda_stream
    if n > 1:
        assert lib.lutkan_model_forward(arr, n, xg.data_ptr(), B, y0.data_ptr(), ptr[0], ws.data_ptr(), ws.numel(), stream) == 0
        plan = lk.lutkan_last_plan()
        assert lib.lutkan_model_forward_or_workspace(arr, n, xg.data_ptr(), B, y1.data_ptr(), ptr[1], C.byref(need), stream) == 0
    else:
        assert lib.lutkan_forward(arr, xg.data_ptr(), B, y0.data_ptr(), ptr[0], ws.data_ptr(), ws.numel(), stream) == 0
        plan = lk.lutkan_last_plan()
        assert lib.lutkan_forward_or_workspace(arr, xg.data_ptr(), B, y1.data_ptr(), ptr[1], C.byref(need), stream) == 0
    if needs:
        assert need.value == room and lk.lutkan_last_plan() == "" and bool((y1 == -7.0).all())
        assert stats[1] is None or int(stats[1].abs().sum()) == 0
    else:
        assert need.value == 0 and lk.lutkan_last_plan() == plan
        assert torch.equal(y0, y1) and (stats[0] is None or torch.equal(stats[0], stats[1]))
    y2 = lk.lutkan_model_forward(layers, xg, stats=stats[2]) if n > 1 else lk.lutkan_forward(layers[0], xg, stats=None if stats[2] is None else stats[2][0])
    assert lk.lutkan_last_plan() == plan and torch.equal(y0, y2) and (stats[0] is None or torch.equal(stats[0], stats[2]))


LONG_SUM_CASES = [
    # seed, d, m, G, boundary, oob, B: 80 inputs per work-group and more; 2, 3, 4 groups of slots; 128, 64 and 32 columns; inputs that end inside a stage
    (951, 121, 129, 5, CLOSED, CLIP_X, 32513),
    (952, 120, 64, 1, HALF_OPEN, ZERO_SPLINE, 66000),
    (953, 123, 20, 4, CLOSED, ZERO_SPLINE, 120001),
    (954, 97, 200, 6, HALF_OPEN, CLIP_X, 20001),
    (955, 98, 40, 9, CLOSED, ZERO_SPLINE, 60001),
    (956, 130, 30, 8, CLOSED, CLIP_X, 60000),
    (957, 81, 128, 13, HALF_OPEN, ZERO_SPLINE, 65001),
    (958, 84, 60, 10, CLOSED, CLIP_X, 65000),
    (959, 83, 9, 11, HALF_OPEN, CLIP_X, 120000),
    (960, 1001, 300, 10, CLOSED, ZERO_SPLINE, 2000),            # in chunks whose sums are added in a second pass
]


def _long_sum_bound(d, G):
    """Of the sum of the terms' magnitudes: 1.3e-6 for basis values, pieces and products (test_bspline_layer_keeps_small_basis_values), and a
    unit in the last place for every addition: the matrix unit's, 8 inputs of one group of slots at a time, the two accumulators' and the chunks'."""
    groups = 2 if G <= 5 else 3 if G <= 9 else 4
    return 1.3e-6 + (d * groups / 8 + 16) * 2.0 ** -23


@pytest.mark.parametrize("case", LONG_SUM_CASES, ids=lambda c: f"seed{c[0]}")
def test_bspline_layer_of_many_inputs(case):
    """Against the oracle in 300 rows, the ends of the batch and rows with a NaN and infinities among them.  Then tables that their owner
    rewrites: scaled by powers of two, all of it or one column, every output is scaled likewise, to the bit; an infinite coefficient of
    the last input shows in the rows on its support."""
    seed, d, m, G, boundary, oob, B = case
    w = random_layer(seed, d, m, G, 2, SYM_INT8, boundary, oob, B, uniform=True)
    s, x = w.layers[0], w.x
    x[3, d // 2] = np.nan
    x[5, :] = np.inf
    x[B - 1, 0] = -np.inf
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob)
    layer = art.bspline_to_device(DEV)
    xg = torch.from_numpy(x).to(DEV)
    _say(f"case many inputs d={d} m={m} G={G} boundary={boundary} oob={oob} B={B}")
    y = lk.bspline_kan_forward(layer, xg)
    plan = lk.lutkan_last_plan()
    assert "slots" in plan and ("sum; " in plan) == (d == 1001), plan
    rng = np.random.Generator(np.random.PCG64(seed))
    rows = np.unique(np.concatenate([np.arange(40), np.arange(B - 40, B), rng.integers(0, B, 300)]))
    ref = oracle.bspline_forward(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.boundary, s.oob, x[rows])
    _assert_close(y.cpu().numpy()[rows], ref, f"many inputs {w.name}")
    held, bound = layer.coef_table.clone(), _long_sum_bound(d, G)
    for exponent in (3, -9, 20, -30):
        layer.coef_table.copy_(held * 2.0 ** exponent)
        scaled = lk.bspline_kan_forward(layer, xg)
        assert torch.equal((scaled * 2.0 ** -exponent).nan_to_num(123.0), y.nan_to_num(123.0)), exponent
    layer.coef_table.copy_(held)
    table = layer.coef_table.view(art.info.coef_n_tiles, d, G + 3, art.info.coef_jt)
    table[0, :, :, 1] *= 2.0 ** -40
    scaled = lk.bspline_kan_forward(layer, xg)
    scaled[:, 1] *= 2.0 ** 40
    assert torch.equal(scaled.nan_to_num(123.0), y.nan_to_num(123.0))
    layer.coef_table.copy_(held)
    table[0, d - 1, 3, 1] = float("inf")
    gather = layer.with_contract(boundary, oob, lk.ALGO_GATHER)
    y, expect = lk.bspline_kan_forward(layer, xg).cpu().numpy()[rows], lk.bspline_kan_forward(gather, xg).cpu().numpy()[rows]
    T, last = s.ext_knots[3:3 + G + 1], x[rows, d - 1]
    masked = (oob == ZERO_SPLINE) & ~((last >= T[0]) & ((last <= T[-1]) if boundary == CLOSED else (last < T[-1])))
    finite = np.where(masked[:, None], np.isfinite(ref.y), np.isfinite(expect))        # (the gather kernel multiplies a masked input's 0 too)
    assert np.array_equal(np.isfinite(y), finite) and np.isinf(y[:, 1]).any()
    assert np.array_equal(np.delete(np.isfinite(y), 1, axis=1), np.delete(np.isfinite(ref.y), 1, axis=1))
    live = np.isfinite(y)
    assert np.all(np.abs(y - ref.y)[live] <= (bound + d * 2.0 ** -21) * ref.A[live])      # (term by term: four products and additions an input)


@pytest.mark.parametrize("exponent", [-20, -30, -40, -60])
@pytest.mark.parametrize("case", [c for c in LONG_SUM_CASES if c[3] > 1], ids=lambda c: f"seed{c[0]}")
def test_bspline_layer_of_many_inputs_keeps_small_coefficients(case, exponent):
    """Every edge has a large coefficient, the first; the others are 2^exponent of it.  Rows whose inputs lie off its support are right
    relative to the sum of their own terms, however small it is beside the table's largest value."""
    seed, d, m, G, boundary, oob, B = case
    w = random_layer(seed, d, m, G, 2, SYM_INT8, boundary, oob, 2, uniform=True)
    s = w.layers[0]
    coef = s.coef.copy()
    coef[:, :, 1:] *= np.float32(2.0 ** exponent)
    coef[:, :, 0] = np.copysign(np.float32(3.9), coef[:, :, 0])
    T = s.ext_knots[3:3 + G + 1]
    rng = np.random.Generator(np.random.PCG64(seed))
    x = np.clip(rng.uniform(T[1], T[-1], size=(B, d)).astype(np.float32), T[1], np.nextafter(T[-1], np.float32(-np.inf)))
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, coef, s.L, s.scheme, s.boundary, s.oob)
    _say(f"case small coefficients d={d} m={m} G={G} 2^{exponent} B={B}")
    y = lk.bspline_kan_forward(art.bspline_to_device(DEV), torch.from_numpy(x).to(DEV))
    assert "slots" in lk.lutkan_last_plan()
    rows = np.unique(rng.integers(0, B, 200))
    ref = oracle.bspline_forward(s.d, s.m, s.G, s.p, s.ext_knots, coef, s.boundary, s.oob, x[rows])
    worst = float(np.max(np.abs(y.cpu().numpy()[rows].astype(np.float64) - ref.y) / ref.A))
    _say(f"  worst {worst:.3g} of the terms, bound {_long_sum_bound(d, G):.3g}")
    assert worst <= _long_sum_bound(d, G), worst


@pytest.mark.parametrize("G", [1, 5, 6, 9, 10, 13])
def test_every_input_of_a_stage_meets_its_own_coefficients(G):
    """The grids at either end of two, three and four groups of slots per input; inputs short of, filling and past a stage of the
    matrix kernel, whose lower lanes take one half of it and upper lanes the other.  All inputs at once, then each alone (the
    others' coefficients are zero: a slot that met a neighbour's shows)."""
    for d in (1, 2, 3, 4, 5, 7, 8, 9, 13, 17):
        w = random_layer(700 + G, d, 5, G, 2, SYM_INT8, CLOSED, CLIP_X, 100, uniform=False)
        s = w.layers[0]
        xg = torch.from_numpy(w.x).to(DEV)
        for only in [None] + list(range(d)):
            coef = s.coef.copy()
            if only is not None:
                coef[np.arange(d) != only] = 0.0
            art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, coef, s.L, s.scheme, s.boundary, s.oob)
            y = lk.bspline_kan_forward(art.bspline_to_device(DEV), xg)
            assert f"slots={8 if G <= 5 else 12 if G <= 9 else 16}; " in lk.lutkan_last_plan(), lk.lutkan_last_plan()
            ref = oracle.bspline_forward(s.d, s.m, s.G, s.p, s.ext_knots, coef, s.boundary, s.oob, w.x)
            _assert_close(y.cpu().numpy(), ref, f"G={G} d={d} only={only}")


def test_bspline_layers_outside_the_matrix_kernel_keep_their_kernels():
    """What the matrix kernel does not serve, and the handful of rows on a large table that it is slower at."""
    for kw, what in ((dict(G=14), "14 segments"), (dict(with_base=True), "spline_component")):
        w = random_layer(921, 12, 40, kw.get("G", 5), 2, SYM_INT8, CLOSED, CLIP_X, 50, with_base=kw.get("with_base", False))
        _check_bspline(w.layers[0], w.x, lk.ALGO_AUTO, what)
        assert lk.lutkan_last_plan().startswith("bspline_locate; bspline_tiled np=") and "slots" not in lk.lutkan_last_plan()
    w = per_input_layer(922, 12, 40, 5, 2, SYM_INT8, CLOSED, CLIP_X, 50)
    s = w.layers[0]
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob, knots_per_input=True)
    lk.bspline_kan_forward(art.bspline_to_device(DEV), torch.from_numpy(w.x).to(DEV))
    assert "slots" not in lk.lutkan_last_plan()
    w = cfg4(B=8)
    s = w.layers[0]
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, 2, s.scheme, s.boundary, s.oob)
    layer, xg = art.bspline_to_device(DEV), torch.from_numpy(w.x).to(DEV)
    lk.bspline_kan_forward(layer, xg[:7])
    assert "bspline_gather" in lk.lutkan_last_plan()
    lk.bspline_kan_forward(layer, xg)
    assert lk.lutkan_last_plan().startswith("bspline_matrix ")


@pytest.mark.parametrize("case", [(995, 37, 70, 5, 300), (996, 130, 200, 10, 90), (997, 9, 6, 5, 5000), (998, 512, 400, 7, 5003)], ids=lambda c: f"seed{c[0]}")
def test_coefficients_that_are_not_finite_reach_the_rows_on_their_support_only(case):
    """The compiler refuses such coefficients; a device table that its owner writes may hold them.  The matrix product multiplies
    every coefficient with every row: 0 * inf must not show.  Against the gather kernel on the same table."""
    seed, d, m, G, B = case
    w = random_layer(seed, d, m, G, 2, SYM_INT8, CLOSED, CLIP_X, B)
    s = w.layers[0]
    art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob)
    layer, other = art.bspline_to_device(DEV), art.bspline_to_device(DEV, lk.ALGO_GATHER)
    xg = torch.from_numpy(w.x).to(DEV)
    clean = lk.bspline_kan_forward(layer, xg)
    info, R = art.info, G + 3
    for held in (layer, other):
        table = held.coef_table.view(torch.float32).view(info.coef_n_tiles, d, R, info.coef_jt)
        table[0, d // 2, 1, 3 % m] = float("inf")
        table[0, 0, R - 2, 1] = float("nan")
        table[-1, d - 1, 2, 0] = float("-inf")
    _say(f"case not finite d={d} m={m} G={G} B={B}")
    y = lk.bspline_kan_forward(layer, xg)
    assert "slots" in lk.lutkan_last_plan()
    expect = lk.bspline_kan_forward(other, xg)
    torch.cuda.synchronize()
    y, expect, clean = y.cpu().numpy(), expect.cpu().numpy(), clean.cpu().numpy()
    assert np.array_equal(np.isfinite(y), np.isfinite(expect)) and 0 < (~np.isfinite(y)).sum() < 3 * B
    assert np.array_equal(y[~np.isfinite(y)], expect[~np.isfinite(expect)], equal_nan=True)
    live = np.isfinite(y)
    assert np.all(np.abs(y - clean)[live] <= 1e-5 * np.sqrt(d) * 4 + 1e-6)


LARGEST_FACTORS = [3.4028234e38, -3.39e38]                 # beyond the largest bf16 value


def _adversarial_factors(rng, n):
    """fp32 values whose lower 16 significand bits weigh most when they are cut off, very small ones, and random ones."""
    special = [1 + 2.0 ** -7 - 2.0 ** -23, 1 + 2.0 ** -8 - 2.0 ** -23, 1 + 2.0 ** -8 + 2.0 ** -16 + 2.0 ** -17, 1 + 2.0 ** -7 - 2.0 ** -16, 2 - 2.0 ** -23,
               1 + 2.0 ** -15 - 2.0 ** -23, 1e-25, -1.0, 1.5]
    return np.concatenate([special, rng.normal(size=n - len(special))]).astype(np.float32)


def _assert_products_like_fp32(got, a, b, last_sum, what):
    """got = a * b for exactly known fp32 a (rows) and b (columns): the dropped piece products (2^-24), the rounding of the five
    small ones' sum (2^-7 of a rounding each) and the result's last sum make (1.1 + last_sum) * 2^-24: 1 where it is an
    addition of the vector ALU, 2 where the matrix unit's accumulator does it, whose rounding mode is not specified (one unit in
    the last place; 2.7 in all is measured, 9.2 with pieces cut by truncation).  Over random factors the errors
    cancel (their mean would be -0.7 * 2^-24 with pieces cut by truncation; 3e5 products leave a deviation of 0.002 * 2^-24)."""
    exact = a.astype(np.float64)[:, None] * b.astype(np.float64)[None, :]
    normal = (np.abs(exact) > 1e-30) & (np.abs(exact) < 3.4e38)
    rel = np.where(normal, got.astype(np.float64) / np.where(normal, exact, 1.0) - 1.0, 0.0) * 2.0 ** 24
    _say(f"case {what}: {int(normal.sum())} products, largest relative error {np.abs(rel).max():.3f} * 2^-24, mean {rel[normal].mean():+.4f}")
    assert np.abs(rel).max() <= 1.1 + last_sum and abs(rel[normal].mean()) <= 0.02


def test_the_pieces_of_products_on_the_matrix_cores_b_spline_layer():
    """A single coefficient c makes the layer's output c times a basis value; the column with c = 1 returns that value as it is.
    A table with coefficients beyond the largest bf16 value is summed term by term."""
    for G, r, largest in ((5, 4, []), (10, 6, []), (10, 6, LARGEST_FACTORS)):
        rng = np.random.Generator(np.random.PCG64(40 + G))
        c = np.concatenate([[1.0], largest, _adversarial_factors(rng, 127 - len(largest))]).astype(np.float32)
        coef = np.zeros((1, len(c), G + 3), np.float32)
        coef[0, :, r] = c
        tau = (-1.0 + (np.arange(G + 7) - 3) * (2.0 / G)).astype(np.float32)
        x = rng.uniform(-1.0, 1.0, (6000, 1)).astype(np.float32)
        art = lk.lutkan_compile(1, len(c), G, 3, tau, coef, 2, SYM_INT8, CLOSED, CLIP_X)
        y = lk.bspline_kan_forward(art.bspline_to_device(DEV), torch.from_numpy(x).to(DEV))
        assert "slots" in lk.lutkan_last_plan()
        y = y.cpu().numpy()
        assert np.isfinite(y).all()
        _assert_products_like_fp32(y[:, 1:], y[:, 0], c[1:], 1.0, f"B-spline G={G}")


def test_the_pieces_of_products_on_the_matrix_cores_base_branch():
    """The base product of a layer whose spline branch is zero and whose first input alone has a base weight."""
    d, m, B = 32, 64, 250000
    rng = np.random.Generator(np.random.PCG64(47))
    c = np.concatenate([[1.0], LARGEST_FACTORS, _adversarial_factors(rng, m - 1 - len(LARGEST_FACTORS))]).astype(np.float32)
    scales = [np.zeros((d, m), np.float32), np.ones((d, m), np.float32), np.ones((d, m), np.float32)]
    scales[0][0] = c
    tau = (-1.0 + (np.arange(12) - 3) * 0.4).astype(np.float32)
    art = lk.lutkan_compile(d, m, 5, 3, tau, np.zeros((d, m, 8), np.float32), 16, SYM_INT8, CLOSED, CLIP_X, edge_scales=tuple(scales))
    x = rng.normal(size=(B, d)).astype(np.float32)
    y = lk.lutkan_forward(art.to_device(DEV), torch.from_numpy(x).to(DEV))
    assert "base_product; " in lk.lutkan_last_plan()
    y = y[:5000].cpu().numpy()
    _assert_products_like_fp32(y[:, 1:], y[:, 0], c[1:], 2.0, "base product")


def _basis64(tau, x, G):
    """All G+3 cubic basis values [len(x), G+3] in extended precision by the Cox-de Boor recursion, positive terms only."""
    tau, x = tau.astype(np.longdouble), x.astype(np.longdouble)
    span = np.clip(np.searchsorted(tau[4:G + 3], x, side="right"), 0, G - 1) + 3
    n = [np.ones_like(x)]
    for q in (1, 2, 3):
        saved, level = np.zeros_like(x), []
        for r in range(q):
            hi, lo = tau[span + r + 1], tau[span + 1 - q + r]
            t = n[r] / (hi - lo)
            level.append(saved + (hi - x) * t)
            saved = (x - lo) * t
        n = level + [saved]
    out = np.zeros((len(x), G + 3), np.longdouble)
    for e in range(4):
        out[np.arange(len(x)), span - 3 + e] = n[e]
    return out


@pytest.mark.parametrize("case", [(5, "uniform", -1.0, 1.0), (8, "uniform", -3.0, 3.0), (10, "uniform", 99.0, 101.0), (13, "uneven", -1.0, 1.0),
                                  (5, "uneven", -2.0, 1.0), (7, "steep", -1.0, 1.0)], ids=lambda c: f"G{c[0]}_{c[1]}")
def test_bspline_layer_keeps_small_basis_values(case):
    """One input and an identity of coefficients return the basis itself: every value, down to those next to the end of a
    function's support, is right relative to itself.  7 roundings of half a unit for the outer functions (each of the three
    factors a subtraction, two products, the factor and its product): 4.2e-7; the middle ones, at least 1/32, have an absolute error
    of 3e-8: 1e-6.  Then coefficients of twelve orders of magnitude: the error stays below 1.3e-6 of the sum of the
    terms' magnitudes (1e-6, and the rounding of four products and their sums)."""
    G, kind, lo, hi = case
    rng = np.random.Generator(np.random.PCG64(G))
    r = np.arange(G + 7) - 3
    tau = (lo + r * ((hi - lo) / G)).astype(np.float32)
    if kind != "uniform":
        gaps = rng.uniform(0.5, 1.5, G + 6) if kind == "uneven" else 10.0 ** rng.uniform(-3.0, 0.0, G + 6)
        grid = np.concatenate([[0.0], np.cumsum(gaps)])
        tau = (lo + (grid - grid[3]) * ((hi - lo) / (grid[3 + G] - grid[3]))).astype(np.float32)
    T = tau[3:3 + G + 1]
    x = [rng.uniform(T[0], T[-1], 4000)]
    for k in range(G):                                    # both ends of every segment, ever closer
        step = (T[k + 1] - T[k]) * 10.0 ** rng.uniform(-6.0, 0.0, 1000)
        x += [T[k] + step, T[k + 1] - step]
    x = np.clip(np.concatenate(x).astype(np.float32), T[0], T[-1])
    expect = _basis64(tau, x, G)
    xg = torch.from_numpy(x[:, None].copy()).to(DEV)
    _say(f"case small basis values G={G} {kind} [{lo}, {hi}] B={len(x)}")

    def forward(coef):
        art = lk.lutkan_compile(1, coef.shape[1], G, 3, tau, coef, 2, SYM_INT8, CLOSED, CLIP_X)
        y = lk.bspline_kan_forward(art.bspline_to_device(DEV), xg)
        plan = lk.lutkan_last_plan()
        assert ("slots" in plan) == (kind != "steep"), plan             # strongly uneven knots stay with the recursion
        torch.cuda.synchronize()
        return y.cpu().numpy().astype(np.longdouble)

    y = forward(np.eye(G + 3, dtype=np.float32)[None])
    live = expect > 1e-30
    assert np.all(y[expect == 0.0] == 0.0)
    worst = float(np.max(np.abs(y - expect)[live] / expect[live]))
    assert worst <= 1e-6, worst
    coef = (rng.choice([-1.0, 1.0], size=(1, 40, G + 3)) * 10.0 ** rng.uniform(-6.0, 6.0, size=(1, 40, G + 3))).astype(np.float32)
    y = forward(coef)
    c = coef[0].astype(np.longdouble).T
    worst = float(np.max(np.abs(y - expect @ c) / (expect @ np.abs(c))))
    assert worst <= 1.3e-6, worst


# ---------------------------------------------------------------- narrow layers in one launch
NARROW_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B, with_base, fp16: tiles of 4, 8, 16, 32 columns; stages of 8 and of 4 slices
    (931, 1000, 4, 10, 16, SYM_INT8, CLOSED, CLIP_X, 5000, False, False),          # inputs split
    (932, 17, 3, 5, 64, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 60000, False, False),  # 8 + 8 + 1 inputs, ragged columns
    (933, 64, 8, 5, 32, ASYM_UINT8, CLOSED, CLIP_X, 40001, False, False),
    (934, 63, 5, 13, 32, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 30000, True, False),    # 13 segments; base branch: stages of 4
    (935, 78, 16, 5, 64, ASYM_UINT8, CLOSED, ZERO_SPLINE, 20011, False, False),
    (936, 90, 13, 10, 64, SYM_INT8, HALF_OPEN, CLIP_X, 20000, False, True),        # long slices: stages of 4; binary16 parameters
    (937, 130, 30, 5, 16, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 30000, False, True),
    (938, 133, 32, 8, 64, SYM_INT8, CLOSED, CLIP_X, 20000, False, False),
    (939, 131, 15, 30, 8, ASYM_UINT8, CLOSED, CLIP_X, 25000, True, False),         # segments searched in steps of eight
    (940, 300, 10, 64, 4, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 3000, False, False),   # the most segments
    (941, 100, 30, 8, 32, SYM_INT8, CLOSED, ZERO_SPLINE, 40001, False, False),     # half stages, two work-groups on a unit
    (942, 100, 30, 8, 32, SYM_INT8, CLOSED, CLIP_X, 40001, False, True),           # the same with binary16 parameters
    (943, 200, 16, 8, 64, ASYM_UINT8, CLOSED, CLIP_X, 2049, False, False),         # too many rows for one wave to walk each
]


@pytest.mark.parametrize("case", NARROW_CASES, ids=lambda c: f"seed{c[0]}")
def test_narrow_layer_in_one_launch(case):
    """Against the oracle and its OOB counters, with NaN, infinite, zero (of both signs) and end-of-domain inputs; rows off
    the 16-byte grid give the same bits."""
    seed, d, m, G, L, scheme, boundary, oob, B, with_base, fp16 = case
    w = random_layer(seed, d, m, G, L, scheme, boundary, oob, B, uniform=(seed % 2 == 0), with_base=with_base)
    s, x = w.layers[0], w.x
    x[7, :] = -0.0
    x[8, :] = 0.0
    x[9, 0] = np.nan
    x[10, d - 1] = np.inf
    x[11, d // 2] = -np.inf
    if with_base:                                          # (an infinite base branch: only its class is defined)
        x[10, d - 1] = x[11, d // 2] = 3.0e38 ** 0.25
    art, ora = _compile_both(s, fp16)
    layer = _device_layer(art, s)
    _say(f"case narrow d={d} m={m} K={G} L={L} scheme={scheme} boundary={boundary} oob={oob} B={B} base={with_base} fp16={fp16}")
    xg = torch.from_numpy(x).to(DEV)
    stats = torch.zeros(2, dtype=torch.int64, device=DEV)
    y = lk.lutkan_forward(layer, xg, stats=stats)
    assert lk.lutkan_last_plan().startswith("narrow split="), lk.lutkan_last_plan()
    shifted = torch.empty(B * d + 1, dtype=torch.float32, device=DEV)[1:].view(B, d).copy_(xg)
    y_shifted = lk.lutkan_forward(layer, shifted)
    torch.cuda.synchronize()
    ref = oracle.lut_forward(ora, s.boundary, s.oob, x, trace=True, edge_scalars=s.edge_scales)
    _assert_close(y.cpu().numpy(), ref, f"narrow {w.name}")
    assert np.array_equal(y.cpu().numpy(), y_shifted.cpu().numpy(), equal_nan=True)
    assert stats.cpu().tolist() == [ref.oob_count, ref.oob_any_rows]


def test_narrow_layer_locates_bit_exactly():
    """Codes q[k][l] = l, alpha_k = 2^k on one input make the output 2^k (l0 + w), exact in fp32: the one-launch kernel's index
    work is the oracle's bit for bit, at the knots, beside them and between."""
    K, L = 12, 16
    for width, (lo, hi) in ((4, (-1.0, 1.0)), (16, (0.0, 3.0))):
        knots = np.linspace(lo, hi, K + 1).astype(np.float32)
        q = np.tile(np.arange(L, dtype=np.uint8), (width, K, 1))
        scale = np.tile((2.0 ** np.arange(K)).astype(np.float32), (width, 1))
        art = lk.lutkan_artifact_from_arrays(1, width, knots, q, scale, np.zeros((width, K), np.float32), CLOSED, CLIP_X)
        rng = np.random.Generator(np.random.PCG64(77))
        x = rng.uniform(lo - 0.1, hi + 0.1, size=(70000, 1)).astype(np.float32)
        near = np.concatenate([knots, np.nextafter(knots, np.float32(-9)), np.nextafter(knots, np.float32(9)), np.float32([0.0, -0.0, 1e-40, -1e-40])])
        x[:near.size, 0] = near
        layer = art.to_device(DEV)
        xg = torch.from_numpy(x).to(DEV)
        y = lk.lutkan_forward(layer, xg)
        assert lk.lutkan_last_plan().startswith("narrow split="), lk.lutkan_last_plan()
        _, k, l0, _, wgt, _ = lk.lutkan_forward_trace(layer, xg)
        expect = (1 << k.long()).double() * (l0.double() + wgt.double())
        # (the running sums carry 2^-24, so a value below 2^-126 * 2^24 -- a weight next to the knot at 0 -- may be flushed)
        flushed = (expect < 2.0 ** -102) & (y.double().abs() <= expect)
        assert torch.equal(torch.where(flushed, expect, y.double()), expect.expand(-1, width))


# Shared grids whose segments are not all between 2^-30 and 2^30 wide, and one whose are.
WIDTH_GRIDS = {
    "subnormal": np.float32([1.0, 2.0, 3.0, 5.0, 9.0]) * np.float32(1e-39),                       # 1 / width is infinite
    "below 2^-30": np.float32([-1.0, 0.0, 1.0, 3.0, 7.0]) * np.float32(2.0 ** -40),
    "above 2^30": np.float32([-5.0, -1.0, 0.0, 2.0, 9.0]) * np.float32(2.0 ** 32),
    "overflowing": np.float32([-3.0e38, 3.0e38, 3.2e38]),                                         # the first width is infinite
    "one of each": np.float32([-3.0e38, -1.0, -1.0 + 2.0 ** -24, 0.0, 1e-39, 1.0, 3.0e38]),
    "2^-30 to 2^30": np.float32([0.0, 2.0 ** -30, 2.0 ** -29, 1.0, 2.0 ** 30]),
}


@pytest.mark.parametrize("grid", WIDTH_GRIDS)
def test_segments_of_any_width_locate_bit_exactly(grid):
    """The revealing table (codes q[k][l] = l, alpha_k = 2^k: the output is 2^k (l0 + w)) on narrow and wide segments, in every kernel
    that locates inputs: at the knots and below the first, where the numerator of Eq. 15 is zero, beside them, between them, and
    with numerators around 2^-90.  Thousands of rows together hold one knot, so that all elements of a thread do."""
    knots = WIDTH_GRIDS[grid]
    K, L, B = knots.size - 1, 16, 70000
    rng = np.random.Generator(np.random.PCG64(78))
    k = rng.integers(0, K, size=B)
    lo, hi = knots[k].astype(np.float64), knots[k + 1].astype(np.float64)
    x = (lo + rng.uniform(size=B) * (hi - lo)).astype(np.float32)
    x[:20000] = np.clip(knots[k[:20000]] + np.ldexp(rng.uniform(1.0, 2.0, size=20000), rng.integers(-100, -80, size=20000)).astype(np.float32), knots[0], knots[-1])
    run = 40000 // (K + 2)
    for n, v in enumerate([np.float32(-3.3e38)] + list(knots)):
        x[20000 + n * run:20000 + (n + 1) * run] = v
    near = np.concatenate([knots, np.nextafter(knots, np.float32(-np.inf)), np.nextafter(knots, np.float32(np.inf))])
    x[:near.size] = near
    with np.errstate(over="ignore"):
        x[~np.isfinite(x - knots[0])] = knots[0]           # (inf / inf: not a number by Eq. 15 itself)
    x = x.reshape(B, 1)
    q = np.tile(np.arange(L, dtype=np.uint8), (1, K, 1))
    scale = (2.0 ** np.arange(K)).astype(np.float32).reshape(1, K)
    ora = SimpleNamespace(d=1, m=1, K=K, L=L, scheme=ASYM_UINT8, knots=knots, q=q, scale=scale, y_min=np.zeros((1, K), np.float32))
    ref = oracle.lut_forward(ora, CLOSED, CLIP_X, x, trace=True)
    z = ref.l0[:, 0].astype(np.float64) + ref.w[:, 0]
    assert np.isfinite(z).all()
    xg = torch.from_numpy(x).to(DEV)

    def check(name, y, first=0):
        assert lk.lutkan_last_plan().startswith(name), lk.lutkan_last_plan()
        got, of = y.cpu().numpy().astype(np.float64), slice(first, first + y.shape[0])
        expect = np.ldexp(z[of], ref.k[of, 0])[:, None]
        # (the running sums carry 2^-24: a z below 2^-126 * 2^24 is subnormal there, flushed or a multiple of 2^-149 * 2^24)
        wrong = (got != expect) & ~((z[of] < 2.0 ** -102)[:, None] & (np.abs(got) <= expect + np.ldexp(2.0 ** -125, ref.k[of, 0])[:, None]))
        row = first + int(np.argmax(wrong.any(axis=1)))
        assert not wrong.any(), f"{name} {y.shape[1]} columns, {grid}: x = {x[row, 0]!r} gives {got[row - first]}, not {expect[row - first]}"

    def layer(m, algo):
        return lk.lutkan_artifact_from_arrays(1, m, knots, np.tile(q, (m, 1, 1)), np.tile(scale, (m, 1)), np.zeros((m, K), np.float32), CLOSED,
                                              CLIP_X).to_device(DEV, algo)

    _say(f"case widths {grid}")
    check("narrow ", lk.lutkan_forward(layer(4, lk.ALGO_AUTO), xg))
    check("narrow ", lk.lutkan_forward(layer(16, lk.ALGO_AUTO), xg))
    check("locate; tiled ", lk.lutkan_forward(layer(1, lk.ALGO_TILED), xg))
    check("locate; gather ", lk.lutkan_forward(layer(1, lk.ALGO_GATHER), xg))
    several = layer(130, lk.ALGO_AUTO)
    for first in range(0, B, 1000):
        check("rows ", lk.lutkan_forward(several, xg[first:first + 1000].contiguous()), first)
    check("locate; tiled ", lk.lutkan_forward(layer(1, lk.ALGO_TILED), xg[:3000].contiguous()))
    one = layer(1, lk.ALGO_AUTO)
    check("chain ", lk.lutkan_chain_forward([one], xg))
    check("locate; ", lk.lutkan_forward_trace(one, xg)[0])


# ---------------------------------------------------------------- a few rows in one launch
ROWS_CASES = [
    # seed, d, m, G, L, scheme, boundary, oob, B, with_base, fp16, per_input: every tile width; one and several rounds of inputs
    (951, 256, 256, 8, 64, SYM_INT8, CLOSED, CLIP_X, 1, False, False, False),
    (952, 257, 300, 7, 48, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 30, False, True, False),     # one input over a round
    (953, 2048, 33, 5, 16, SYM_INT8, CLOSED, ZERO_SPLINE, 17, False, False, False),        # the most inputs
    (954, 65, 70, 13, 32, ASYM_UINT8, CLOSED, CLIP_X, 500, True, False, False),            # four rows per work-group; 13 segments
    (955, 300, 128, 5, 32, SYM_INT8, HALF_OPEN, CLIP_X, 203, False, False, True),          # one knot vector per input
    (956, 1500, 3, 6, 16, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 9, True, False, False),      # 4-column tile
    (957, 1100, 30, 5, 64, SYM_INT8, CLOSED, CLIP_X, 20, False, True, False),              # binary16 parameter rows
    (958, 600, 10, 64, 4, ASYM_UINT8, CLOSED, ZERO_SPLINE, 33, False, True, True),
    (959, 1030, 6, 5, 32, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 5, False, False, False),       # 8-column tile
]


ROUND_CASES = [
    # as above: no group with more than one input, than two, one input over; more work-groups than compute units, odd numbers of rounds
    (961, 64, 130, 8, 64, SYM_INT8, CLOSED, CLIP_X, 3, False, False, False),
    (962, 128, 70, 5, 32, ASYM_UINT8, HALF_OPEN, ZERO_SPLINE, 5, True, False, False),
    (963, 129, 70, 5, 32, SYM_INT8, CLOSED, ZERO_SPLINE, 5, False, True, False),
    (964, 16, 300, 6, 48, ASYM_UINT8, CLOSED, CLIP_X, 703, False, False, False),
    (965, 33, 200, 9, 32, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 901, True, False, False),
    (966, 100, 100, 5, 64, ASYM_UINT8, CLOSED, CLIP_X, 1021, False, True, False),
    (967, 47, 260, 7, 16, SYM_INT8, HALF_OPEN, CLIP_X, 600, False, False, True),
    (968, 1, 500, 5, 32, ASYM_UINT8, CLOSED, ZERO_SPLINE, 160, False, False, False),
    (969, 1211, 64, 5, 16, SYM_INT8, CLOSED, CLIP_X, 1025, False, False, False),           # the most inputs whose records let two share a unit
    (970, 1212, 64, 5, 16, SYM_INT8, HALF_OPEN, ZERO_SPLINE, 1025, False, False, False),
]


def test_rounds_of_two_where_two_work_groups_share_a_compute_unit():
    """The kernel for a few rows: two inputs a round where more work-groups than compute units wait and the LDS holds two of them, or where
    no group has more; four else."""
    for d, m, B, depth in ((128, 64, 9, 2), (256, 64, 1020, 4), (256, 64, 1025, 2), (1211, 64, 1025, 2), (1212, 64, 1025, 4), (1220, 64, 1030, 4)):
        w = random_layer(971, d, m, 5, 16, SYM_INT8, CLOSED, CLIP_X, B)
        s = w.layers[0]
        art = lk.lutkan_compile(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.L, s.scheme, s.boundary, s.oob)
        lk.lutkan_forward(art.to_device(DEV), torch.from_numpy(w.x).to(DEV))
        plan = lk.lutkan_last_plan()
        assert plan.startswith("rows wpr=") and plan.endswith(f" depth={depth}; "), (d, m, B, plan)


@pytest.mark.parametrize("case", [
    # d, m, G, L, scheme, B, with_base, per_input, the plan's first clause: narrow inputs, and many with knots each, by the passes, others and launches of a round or so in one
    (1, 272, 5, 64, SYM_INT8, 1104, False, False, "locate; tiled"), (2, 976, 8, 32, ASYM_UINT8, 290, False, False, "locate; tiled"),
    (9, 298, 5, 32, ASYM_UINT8, 1952, False, False, "locate; tiled"), (34, 1000, 12, 64, SYM_INT8, 870, False, False, "locate; tiled"),
    (793, 28, 12, 64, SYM_INT8, 1863, False, True, "locate; tiled"), (123, 461, 3, 64, SYM_INT8, 534, False, True, "rows"),
    (1, 357, 5, 64, SYM_INT8, 338, False, False, "rows"), (100, 200, 5, 64, SYM_INT8, 1000, False, False, "rows"), (86, 249, 5, 32, ASYM_UINT8, 766, True, False, "rows"),
], ids=lambda c: f"{c[0]}-{c[1]}x{c[5]}")
def test_narrow_inputs_run_by_the_passes(case):
    """Which launches of more work-groups than compute units the kernel for a few rows takes; outputs against the oracle either way."""
    d, m, G, L, scheme, B, with_base, per_input, clause = case
    w = (per_input_layer if per_input else random_layer)(972, d, m, G, L, scheme, CLOSED, CLIP_X, B, with_base=with_base)
    art, ora = _compile_both(w.layers[0])
    y = lk.lutkan_forward(_device_layer(art, w.layers[0]), torch.from_numpy(w.x).to(DEV))
    assert lk.lutkan_last_plan().startswith(clause), lk.lutkan_last_plan()
    _assert_close(y.cpu().numpy(), oracle.lut_forward(ora, CLOSED, CLIP_X, w.x, trace=True, edge_scalars=w.layers[0].edge_scales), str(case))


@pytest.mark.parametrize("case", ROWS_CASES + ROUND_CASES, ids=lambda c: f"seed{c[0]}")
def test_few_rows_in_one_launch(case):
    """Against the oracle and its OOB counters, with NaN, infinite and zero (of both signs) inputs."""
    seed, d, m, G, L, scheme, boundary, oob, B, with_base, fp16, per_input = case
    make = per_input_layer if per_input else random_layer
    w = make(seed, d, m, G, L, scheme, boundary, oob, B, with_base=with_base)
    s, x = w.layers[0], w.x
    if B > 8:
        x[1, :] = -0.0
        x[2, 0] = np.nan
        if not with_base:                                  # (an infinite base branch: only its class is defined)
            x[3, d - 1] = np.inf
            x[B - 1, d // 2] = -np.inf
    art, ora = _compile_both(s, fp16)
    layer = _device_layer(art, s)
    _say(f"case rows d={d} m={m} K={G} L={L} scheme={scheme} boundary={boundary} oob={oob} B={B} base={with_base} fp16={fp16} per_input={per_input}")
    xg = torch.from_numpy(x).to(DEV)
    stats = torch.zeros(2, dtype=torch.int64, device=DEV)
    y = lk.lutkan_forward(layer, xg, stats=stats)
    assert lk.lutkan_last_plan().startswith("rows wpr="), lk.lutkan_last_plan()
    y_again = lk.lutkan_forward(layer, xg)
    torch.cuda.synchronize()
    ref = oracle.lut_forward(ora, s.boundary, s.oob, x, trace=True, edge_scalars=s.edge_scales)
    _assert_close(y.cpu().numpy(), ref, f"rows {w.name}")
    assert np.array_equal(y.cpu().numpy(), y_again.cpu().numpy(), equal_nan=True)
    assert stats.cpu().tolist() == [ref.oob_count, ref.oob_any_rows]


# ---------------------------------------------------------------- the two phases as separate calls
TWO_PHASE_CASES = [
    # seed, d, m, G, L, scheme, B, with_base: batches whose launch plans read fewer rows than records are laid out for
    (981, 40, 70, 5, 16, SYM_INT8, 70, False),
    (982, 33, 130, 8, 32, ASYM_UINT8, 300, False),
    (983, 300, 64, 6, 16, SYM_INT8, 1, False),
    (984, 65, 20, 7, 32, ASYM_UINT8, 1300, False),
    (985, 40, 70, 5, 16, ASYM_UINT8, 257, True),
]


@pytest.mark.parametrize("case", TWO_PHASE_CASES, ids=lambda c: f"seed{c[0]}")
def test_locate_and_edges_as_separate_calls(case):
    """locate, then edges, against the oracle, and bit for bit what one call on the same kernels returns.  Where a record
    of a separate phase lies follows from B alone: a phi layer's records serve edge phases of every algo and table form."""
    seed, d, m, G, L, scheme, B, with_base = case
    w = random_layer(seed, d, m, G, L, scheme, HALF_OPEN, ZERO_SPLINE, B, uniform=False, with_base=with_base)
    s, x = w.layers[0], w.x
    art, ora = _compile_both(s)
    xg = torch.from_numpy(x).to(DEV)
    ref = oracle.lut_forward(ora, s.boundary, s.oob, x, trace=True, edge_scalars=s.edge_scales)
    forms = [("auto", _device_layer(art, s)), ("gather", _device_layer(art, s, lk.ALGO_GATHER)), ("tiled", _device_layer(art, s, lk.ALGO_TILED))]
    if art.info.jt == 64 and not with_base:
        forms += [(f"wide{cb}", _device_layer(art, s, lk.ALGO_TILED_WIDE, wide=cb)) for cb in (2, 4)]
    nbytes = max(lk.lutkan_forward_workspace_bytes(layer, B) for _, layer in forms)
    for first, located in forms:
        for second, summed in forms:
            if with_base and first != second:          # (what a record holds then depends on algo)
                continue
            _say(f"case two phases d={d} m={m} L={L} scheme={scheme} B={B} base={with_base}: {first} then {second}")
            ws = torch.zeros(nbytes, dtype=torch.uint8, device=DEV)
            y = torch.empty((B, m), dtype=torch.float32, device=DEV)
            lk.lutkan_forward_locate(located, xg, ws)
            lk.lutkan_forward_edges(summed, B, y, ws)
            whole = lk.lutkan_forward(summed, xg)
            torch.cuda.synchronize()
            _assert_close(y.cpu().numpy(), ref, f"{first} then {second}")
            if second != "auto":
                assert torch.equal(y, whole)


@pytest.mark.parametrize("case", [(991, 256, 200, 64), (992, 300, 10, 3000), (993, 64, 8, 70000), (994, 70, 300, 30)], ids=lambda c: f"seed{c[0]}")
def test_outputs_that_lie_partly_over_the_inputs(case):
    """y starts inside x, or x inside y: every kernel of such a call has read what it needs before y is written.  The same
    layers apart run in one launch that reads x to its end."""
    seed, d, m, B = case
    w = random_layer(seed, d, m, 5, 16, SYM_INT8, CLOSED, ZERO_SPLINE, B)
    s, x = w.layers[0], w.x
    art, ora = _compile_both(s)
    layer, spline = _device_layer(art, s), art.bspline_to_device(DEV)
    ref = oracle.lut_forward(ora, s.boundary, s.oob, x, trace=True)
    refb = oracle.bspline_forward(s.d, s.m, s.G, s.p, s.ext_knots, s.coef, s.boundary, s.oob, x)
    xg = torch.from_numpy(x).to(DEV)
    lk.lutkan_forward(layer, xg)
    assert lk.lutkan_last_plan().startswith(("rows ", "narrow "))
    for what, at_x, at_y in (("y in x", 0, B * d // 2 & ~3), ("x in y", B * m // 2 & ~3, 0), ("one row apart", 0, 4)):
        _say(f"case overlap {what}: d={d} m={m} B={B}")
        buf = torch.zeros(max(at_x + B * d, at_y + B * m), dtype=torch.float32, device=DEV)
        xv, yv = buf[at_x:at_x + B * d].view(B, d), buf[at_y:at_y + B * m].view(B, m)
        xv.copy_(xg)
        stats = torch.zeros(2, dtype=torch.int64, device=DEV)
        lk.lutkan_forward(layer, xv, yv, stats=stats)
        torch.cuda.synchronize()
        _assert_close(yv.cpu().numpy(), ref, what)
        assert stats.cpu().tolist() == [ref.oob_count, ref.oob_any_rows]
        xv.copy_(xg)
        lk.bspline_kan_forward(spline, xv, yv)
        torch.cuda.synchronize()
        _assert_close(yv.cpu().numpy(), refb, "bspline " + what)


@pytest.mark.parametrize("workload,batch", [("cfg3_L64_sym", 256), ("cfg2", 20000), ("cfg5_closed_clip_x", 64)])
def test_bench_times_the_calls_that_run_in_one_launch(workload, batch):
    """bench.py takes a call apart into its phases only where it has two; the layers of these workloads run on the rows, narrow
    and chain kernels."""
    import bench
    rec = bench.run_workload(bench.Rig(probes=False), workload, steps=2, warmup=1, batch=batch, bspline=False, cpu_baseline=False)
    named = [k["kernel"] for k in rec["kernels"]]
    assert any(k in ("lutkan_rows_kernel", "lutkan_narrow_kernel") for k in named), named
    assert all(k["ms"] > 0 for k in rec["kernels"]) and rec["roofline"]["terms"]["work"]["hbm"] > 0


def test_calls_run_on_torchs_current_stream():
    """The stream handle that a call gets is the current stream's, on the default stream and on others, and work queued
    there before the call is seen by it."""
    from paper_2601_03332_amd import binding
    dev = torch.empty(1, device=DEV).device
    assert binding._stream(dev) == torch.cuda.current_stream(dev).cuda_stream
    w = random_layer(971, 40, 70, 5, 16, SYM_INT8, CLOSED, CLIP_X, 64)
    layer = _device_layer(_compile_both(w.layers[0])[0], w.layers[0])
    xg = torch.from_numpy(w.x).to(DEV)
    expect = lk.lutkan_forward(layer, xg)
    torch.cuda.synchronize()
    side = torch.cuda.Stream(dev)
    with torch.cuda.stream(side):
        assert binding._stream(dev) == side.cuda_stream == torch.cuda.current_stream(dev).cuda_stream
        late = torch.zeros_like(xg)
        for _ in range(20):
            late.add_(1.0)
        late.copy_(xg)
        y = lk.lutkan_forward(layer, late)
    side.synchronize()
    assert binding._stream(dev) == torch.cuda.current_stream(dev).cuda_stream
    assert torch.equal(y, expect)


class _Intercepts(torch.overrides.TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def test_native_calls_take_the_plain_case_and_leave_the_rest_to_the_general_path():
    """A call without optional arguments in native code: bit for bit the general path's output, with and without a workspace, on the
    current stream, for one layer, a network and the B-spline layer; None, with nothing done, for whatever is not plain."""
    from paper_2601_03332_amd import binding
    native = binding._native_calls()
    w = random_layer(981, 40, 50, 5, 16, SYM_INT8, CLOSED, CLIP_X, 3000)
    arts = [_compile_both(s)[0] for s in (w.layers[0], random_layer(982, 50, 7, 6, 16, SYM_INT8, CLOSED, CLIP_X, 1).layers[0])]
    layers, spline = [a.to_device(DEV) for a in arts], arts[0].bspline_to_device(DEV)
    x = torch.from_numpy(w.x).to(DEV)
    side = torch.cuda.Stream()
    for B in (0, 1, 60, 3000):
        _say(f"case native calls B={B}")
        xb = x[:B].clone()
        side.wait_stream(torch.cuda.current_stream())
        for call, general, held in ((native.lut_forward, lk.lutkan_forward, layers[0]), (native.lut_model_forward, lk.lutkan_model_forward, layers),
                                    (native.spline_forward, lk.bspline_kan_forward, spline)):
            m = held[-1].m if held is layers else held.m
            expect = general(held, xb, y=torch.full((B, m), 7.0, device=DEV))
            plan = lk.lutkan_last_plan()
            assert torch.equal(call(held, xb), expect) and (B == 0 or lk.lutkan_last_plan() == plan)
            with torch.cuda.stream(side):
                y = general(held, xb)
            side.synchronize()
            assert torch.equal(y, expect) and not y.requires_grad
            other = held if held is not layers else tuple(held)
            assert torch.equal(call(other, torch.nn.Parameter(xb)), expect)
            subclass = xb.as_subclass(type("Sub", (torch.Tensor,), {}))
            with _Intercepts():
                assert call(held, xb) is None and torch.equal(general(held, xb), expect)
            for bad in (subclass, xb[:, 1:], xb.double(), xb.cpu(), xb.t(), xb[None], xb.numel(), None):
                assert call(held, bad) is None
            if B > 1:
                strided = torch.empty(B, 2 * xb.shape[1], device=DEV)[:, ::2]
                assert call(held, strided) is None
                with pytest.raises(lk.LutKanError, match="contiguous"):
                    general(held, strided)
            with pytest.raises(lk.LutKanError, match="shape"):
                general(held, xb[:, 1:])
    assert native.lut_forward(spline, x) is None and native.spline_forward(layers[0], x) is None
    assert native.lut_model_forward([], x) is None and native.lut_model_forward([layers[1], layers[0]], x) is None
    broken = layers[0].with_contract(CLOSED, CLIP_X)
    broken.c.d = 0                                         # the library refuses it: the general path says why
    assert native.lut_forward(broken, x) is None
    with pytest.raises(lk.LutKanError, match="lutkan_forward"):
        lk.lutkan_forward(broken, x)


def test_native_calls_leave_deferred_and_traced_operators_to_the_general_path():
    """Inference mode is the plain case; fake tensors, functional transforms, functionalisation, tracing and dispatch modes are not."""
    from paper_2601_03332_amd import binding
    from torch._subclasses import FakeTensorMode
    from torch.utils._python_dispatch import TorchDispatchMode
    native = binding._native_calls()
    w = random_layer(984, 12, 20, 5, 16, SYM_INT8, CLOSED, CLIP_X, 40)
    art, _ = _compile_both(w.layers[0])
    layer, x = art.to_device(DEV), torch.from_numpy(w.x).to(DEV)
    calls = [(native.lut_forward, lk.lutkan_forward, layer), (native.lut_model_forward, lk.lutkan_model_forward, [layer]),
             (native.spline_forward, lk.bspline_kan_forward, art.bspline_to_device(DEV))]
    expect = [general(held, x) for _, general, held in calls]

    with torch.inference_mode():
        for (call, general, held), y in zip(calls, expect):
            for got in (call(held, x), call(held, x.clone()), general(held, x, y=torch.empty_like(y))):
                assert torch.equal(got, y) and got.is_inference()

    class Passes(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    taken = []

    def ask(t):
        taken.extend(call(held, t if t.dim() == 2 else t[None]) for call, _, held in calls)
        return t + 1.0

    with FakeTensorMode(allow_non_fake_inputs=True) as mode:
        ask(mode.from_tensor(x))
        ask(x)
    with Passes():
        ask(x)
        assert torch.equal(lk.lutkan_forward(layer, x), expect[0])            # the general path serves it
    torch.func.vmap(ask)(x)
    torch.func.grad(lambda t: ask(t).sum())(x)
    torch.func.jvp(ask, (x,), (torch.ones_like(x),))
    torch.func.functionalize(ask)(x)
    torch.jit.trace(ask, (x,), check_trace=False)
    assert len(taken) == 3 * 8 and all(y is None for y in taken), [y is None for y in taken]
    for (call, _, held), y in zip(calls, expect):                           # and nothing of it is left behind
        assert torch.equal(call(held, x), y)
