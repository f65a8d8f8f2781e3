"""Parity at the sizes where a kernel's tiling or a dispatch rule can go wrong:
remainders of tiles, the smallest and the largest of a range, the lines
between two paths.  Every case runs the whole stage against the oracle."""

import numpy as np
import pytest

from oracle import pulse_oracle as O
from oracle import transformer_oracle as TO
from paper_2606_19163_amd import configs, synth
from paper_2606_19163_amd import tstage as TS

from gpu_util import compare, log, rel_l2, run_gpu

pytestmark = pytest.mark.gpu


def _pair(batch, h, w, c, groups, temb, dtype, n):
    d = configs._pair_stage(batch, h, c, groups, temb, dtype, n_blocks=n)
    return dict(d, width=w)


def _parity(desc, seed, label):
    log(f"case {label}: B={desc['batch']} {desc['height']}x{desc['width']} seed={seed}")
    params, b = synth.make_all(desc, seed)
    gpu, _ = run_gpu(desc, params, b)
    f = lambda d: {k: np.asarray(v, np.float64) for k, v in d.items()}
    p, bb = f(params), f(b)
    ref = O.stage_run(desc, p, bb["x"], bb["u"], bb["temb"], bb["g_enc"], bb["g_dec"])
    compare(desc, gpu, ref, label=label)


@pytest.mark.parametrize("dtype,c", [(configs.F32, 32), (configs.BF16, 96)])
def test_refresh_job_tables(dtype, c):
    """5 + 5 blocks make 36 weight-copy jobs (two tables of 32), with rows
    and columns that are not multiples of the 64 x 64 tile."""
    _parity(_pair(1, 5, 3, c, 8, 64, dtype, 5), 21, f"refresh-{dtype}")


# fp32 and 32-channel bf16 stages with the tiles and K splits that their rules
# pick (test_tiles_forced runs each tile whatever the rules say): remainders in
# rows and columns, images smaller than a tile
CONV_EDGES = [
    (configs.F32, 1, 3, 5, 96, 32, 1), (configs.F32, 2, 33, 31, 64, 16, 1),
    (configs.F32, 4, 48, 48, 160, 32, 1), (configs.F32, 1, 16, 16, 224, 32, 1),
    (configs.BF16, 1, 7, 3, 32, 8, 1), (configs.BF16, 3, 27, 45, 96, 32, 1),
    (configs.BF16, 2, 13, 11, 288, 32, 1), (configs.BF16, 7, 61, 59, 160, 32, 1),
    (configs.BF16, 9, 57, 64, 224, 32, 1), (configs.BF16, 2, 16, 16, 352, 32, 1),
]


@pytest.mark.parametrize("dtype,batch,h,w,c,groups,n", CONV_EDGES,
                         ids=[f"{d}-{b}x{h}x{w}x{c}" for d, b, h, w, c, _, _ in CONV_EDGES])
def test_conv_tiles(dtype, batch, h, w, c, groups, n):
    _parity(_pair(batch, h, w, c, groups, 64, dtype, n), 22, f"{dtype} {batch}x{h}x{w}x{c}")


# grids that do not fill the GPU: every small tile and K grouping is picked by
# some conv of these stages, with ragged rows, K splits whose last split and
# last K group are shorter, and images smaller and larger than a tile
SMALL = [(1, 3, 5, 64, 1), (2, 8, 8, 640, 1), (1, 16, 16, 320, 2), (3, 9, 7, 448, 1),
         (2, 24, 24, 128, 1), (1, 40, 36, 192, 1), (4, 16, 16, 512, 1)]


@pytest.mark.parametrize("batch,h,w,c,n", SMALL, ids=[f"{b}x{h}x{w}x{c}" for b, h, w, c, _ in SMALL])
def test_small_grids(batch, h, w, c, n):
    _parity(_pair(batch, h, w, c, 32, 64, configs.BF16, n), 23, f"small {batch}x{h}x{w}x{c}")


@pytest.mark.parametrize("tile", [4, 5, 6, 7])
@pytest.mark.parametrize("batch,h,w", [(2, 12, 10), (2, 16, 8)])
def test_small_tiles_forced(monkeypatch, tile, batch, h, w):
    """Each small tile on every conv of a stage: K shorter than its groups'
    pipeline (the 1x1 shortcut), epilogue statistics and GroupNorm-backward
    sums (128-pixel images hold whole tiles) and ragged rows."""
    monkeypatch.setenv("PULSE_CONV_TILE", str(tile))
    monkeypatch.setenv("PULSE_CONV_KSPLIT_MAX", "1")
    _parity(_pair(batch, h, w, 128, 32, 64, configs.BF16, 1), 24, f"tile{tile}")


# the 32-channel tiles (128 x 160, 128 x 128, 64 x 96), the fp32 ones (64 x 64,
# 64 x 32, 32 x 32) and the 64-channel ones of small grids
@pytest.mark.parametrize("split", [1, 16])
@pytest.mark.parametrize("batch,h,w", [(2, 13, 11), (2, 16, 8)])
@pytest.mark.parametrize("dtype,tile,c", [(configs.BF16, 8, 160), (configs.BF16, 9, 160),
                                          (configs.BF16, 10, 160), (configs.F32, 11, 96),
                                          (configs.F32, 12, 96), (configs.F32, 13, 96)]
                         + [(configs.BF16, t, 192) for t in (4, 5, 6, 7)])
def test_tiles_forced(monkeypatch, dtype, tile, c, batch, h, w, split):
    """Each of these tiles on every conv of a stage, in one K split (with
    epilogue statistics where 128-pixel images hold whole tiles) and in the
    several that such small grids get, on ragged rows and columns."""
    monkeypatch.setenv("PULSE_CONV_TILE", str(tile))
    monkeypatch.setenv("PULSE_CONV_KSPLIT_MAX", str(split))
    _parity(_pair(batch, h, w, c, 32, 64, dtype, 1), 24, f"tile{tile} splits<={split}")


# bias gradients inside the weight GEMMs: fewer K-steps than column tiles
# (8 x 8 images) and more, the 320-row tile (320 channels; it takes no others,
# as its rows divide them), 128-row tiles with rows past the end (448 and 288)
# and the fp32 loop; their sums go to two biases in decoder blocks
BIAS = [(configs.BF16, 1, 8, 8, 320), (configs.BF16, 2, 33, 20, 448), (configs.BF16, 1, 20, 33, 288),
        (configs.F32, 1, 40, 17, 96)]


@pytest.mark.parametrize("dtype,batch,h,w,c", BIAS, ids=[f"{d}-{b}x{h}x{w}x{c}" for d, b, h, w, c in BIAS])
def test_bias_gradients(dtype, batch, h, w, c):
    _parity(_pair(batch, h, w, c, 32, 64, dtype, 1), 25, f"bias {dtype} {batch}x{h}x{w}x{c}")


def test_fp32_weight_gradient_sums():
    """Long pixel sums of an fp32 weight gradient (24576 pixels of 192
    channels): the shortcut's, over the decoder input and the output gradient,
    which are exact inputs.  Values added one by one in fp32 are off by 0.45 u
    sqrt(n / 2) of their sum, u = 2^-24 (0.45 u: a rounding's root mean
    square): 3.0e-7 for the 256 pixels of one accumulator and 1.9e-7 for 96
    such sums, 3.5e-7 together; twice that is allowed.  One accumulator over a
    pixel split of 4096 to 8192 is off by 1.2e-6 to 1.7e-6."""
    desc = _pair(8, 48, 64, 192, 32, 64, configs.F32, 1)
    log("case fp32 sums: B=8 48x64x192 seed=27")
    params, b = synth.make_all(desc, 27)
    gpu, _ = run_gpu(desc, params, b, want_cache=False)
    u = np.asarray(b["u"], np.float64).reshape(-1, 192)
    g = np.asarray(b["g_dec"], np.float64).reshape(-1, 192)
    e = rel_l2(gpu["grads"]["dec0.Ws"][:, :192], g.T @ u)
    log(f"  fp32 sums dec0.Ws = {e:.3e}")
    assert e < 7e-7, e


# LayerNorm backward by width: rows in one to four waves of 512 channels, the
# last one partly empty (576, 1088, 1600) and full (2048), fewer tokens than
# blocks allowed and more (576 over 512 blocks); three blocks per half write
# the column-sum buffers of the first parity twice
@pytest.mark.parametrize("batch,tokens,heads,n", [(1, 64, 9, 1), (9, 64, 17, 1), (1, 64, 25, 1),
                                                  (9, 64, 32, 1), (2, 64, 2, 3)])
def test_layernorm_backward_widths(batch, tokens, heads, n):
    d = configs._tstage(batch, tokens, 64 * heads, heads, n, n)
    d["mlp"] = 1
    log(f"case LayerNorm backward: B={batch} tokens={tokens} heads={heads} blocks={n}+{n}")
    p, b = synth.make_tstage(d, 28)
    ref = TO.tstage_run(d, p, b["x"], b["u"], b["g_enc"], b["g_dec"])
    st = TS.TStage(d)
    st.set_params(p)
    dev = {k: st.to_dev(v) for k, v in b.items()}
    st.zero_grads()
    got = dict(y_enc=st.forward(TS.ENC, 0, dev["x"]), y_dec=st.forward(TS.DEC, 0, dev["u"]))
    got["du"] = st.backward(TS.DEC, 0, dev["g_dec"])
    got["dx"] = st.backward(TS.ENC, 0, dev["g_enc"])
    got = {k: v.float().cpu().numpy() for k, v in got.items()}
    got.update(st.grads_dict())
    want = dict(ref["grads"], **{k: ref[k] for k in ("y_enc", "y_dec", "du", "dx")})
    errs = {k: rel_l2(got[k], v) for k, v in want.items()}
    worst = max(errs, key=errs.get)
    log(f"  worst {worst} = {errs[worst]:.3e}")
    bad = {k: e for k, e in errs.items() if not e < 2e-2}  # bf16 values, fp32 sums
    assert not bad, bad


# Attention backward with p and ds in registers: from 2048 tokens on, and from
# 512 blocks on beyond 256 tokens; both lengths end in half a 128-key chunk.
@pytest.mark.parametrize("batch,tokens,heads", [(1, 2112, 2), (14, 320, 8)])
def test_attention_backward_in_registers(batch, tokens, heads):
    import torch
    d = configs._tstage(batch, tokens, 64 * heads, heads, 1, 1)
    d["mlp"] = 2
    p, b = synth.make_tstage(d, 26)
    log(f"case attention backward: B={batch} tokens={tokens} heads={heads}")
    ref = TO.tstage_run(d, p, b["x"], b["u"], b["g_enc"], b["g_dec"])
    st = TS.TStage(d)
    st.set_params(p)
    dev = {k: st.to_dev(v) for k, v in b.items()}
    runs = []
    for _ in range(2):
        st.zero_grads()
        st.forward(TS.ENC, 0, dev["x"])
        st.forward(TS.DEC, 0, dev["u"])
        du = st.backward(TS.DEC, 0, dev["g_dec"]).clone()
        dx = st.backward(TS.ENC, 0, dev["g_enc"]).clone()
        torch.cuda.synchronize()
        runs.append(dict(st.grads_dict(), du=du.float().cpu().numpy(),
                         dx=dx.float().cpu().numpy()))
    want = dict(ref["grads"], du=ref["du"], dx=ref["dx"])
    for k, v in want.items():
        assert np.array_equal(runs[0][k], runs[1][k]), k  # reruns are bitwise identical
        e = rel_l2(runs[0][k], v)
        assert e < 2e-2, (k, e)  # bf16 activations and weights, fp32 sums
