"""GPU parity: dit_block_forward / dit_block_mlp against the oracle.

Tolerances. The block contract is a normwise max relative error of 2e-2 on the
block output (bf16 storage, fp32 accumulation). The branch delta (out - in)
is gated too, at 2e-2 of max|delta| plus the unavoidable rounding of the bf16
output itself (half an ulp, <= 2^-8 max|out|). The fp32 configuration is held
to 1e-4."""
import dataclasses

import numpy as np
import pytest
import torch

import seeded_inputs as si
from oracle import dit_oracle as O
from tests.conftest import weights_f64
from tests.gpu_util import block_cfg, dev, host64, rel_err, upload_block

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    from paper_2606_19004_amd import ditstep
    return ditstep


def tol(cfg):
    return 2e-2 if cfg.dtype == "bf16" else 1e-4


def check(cfg, got, ref, inp):
    t = tol(cfg)
    assert rel_err(got, ref) <= t, rel_err(got, ref)
    floor = 2.0 ** -8 * np.max(np.abs(ref)) if cfg.dtype == "bf16" else 0.0
    derr = np.max(np.abs((got - inp) - (ref - inp)))
    assert derr <= t * np.max(np.abs(ref - inp)) + floor, (derr, np.max(np.abs(ref - inp)), floor)


def run_block(d, cfg, inp, mlp_only=False):
    c = block_cfg(d, cfg)
    w = upload_block(inp["weights"], cfg.dtype)
    bw = d.block_weights(w["img"], w["txt"])
    temb = dev(inp["temb"])
    xi, xt = dev(inp["x_img"], cfg.dtype), dev(inp["x_txt"], cfg.dtype)
    ws = d.workspace(d.dit_block_workspace_bytes(c, cfg.batch))
    (d.dit_block_mlp if mlp_only else d.dit_block_forward)(c, bw, temb, xi, xt, ws)
    torch.cuda.synchronize()
    return host64(xi), host64(xt), (c, bw, temb, xi, xt, ws, w)


@pytest.mark.parametrize("name", ["tiny_f32", "small_bf16", "small_bf16_d64"])
def test_block_small_full_compare(d, name):
    cfg = si.CONFIGS[name]
    inp = si.block_inputs(cfg)
    gi, gt, _ = run_block(d, cfg, inp)
    w64 = weights_f64(inp["weights"], cfg.dtype)
    xi, xt = si.as_f64(inp["x_img"], cfg.dtype), si.as_f64(inp["x_txt"], cfg.dtype)
    ri, rt = O.block_forward(cfg, w64, inp["temb"].astype(np.float64), xi, xt)
    check(cfg, gi, ri, xi)
    check(cfg, gt, rt, xt)


@pytest.mark.parametrize("name", ["small_bf16", "tiny_f32"])
def test_block_rope_off_and_no_text(d, name):
    cfg = dataclasses.replace(si.CONFIGS[name], rope=False)
    inp = si.block_inputs(cfg)
    gi, gt, _ = run_block(d, cfg, inp)
    w64 = weights_f64(inp["weights"], cfg.dtype)
    xi, xt = si.as_f64(inp["x_img"], cfg.dtype), si.as_f64(inp["x_txt"], cfg.dtype)
    ri, rt = O.block_forward(cfg, w64, inp["temb"].astype(np.float64), xi, xt)
    check(cfg, gi, ri, xi)
    # no text tokens at all: image-only self-attention
    cfg0 = dataclasses.replace(si.CONFIGS[name], n_txt=0)
    inp0 = si.block_inputs(cfg0)
    gi0, _, _ = run_block(d, cfg0, inp0)
    w0 = weights_f64(inp0["weights"], cfg0.dtype)
    xi0 = si.as_f64(inp0["x_img"], cfg0.dtype)
    ri0, _ = O.block_forward(cfg0, w0, inp0["temb"].astype(np.float64), xi0, np.zeros((cfg0.batch, 0, cfg0.hidden)))
    check(cfg0, gi0, ri0, xi0)


def test_block_adaln_zero_identity_bit_exact(d):
    cfg = si.CONFIGS["small_bf16"]
    inp = si.block_inputs(cfg)
    D = cfg.hidden
    for s in ("img", "txt"):
        for chunk in (2, 5):    # gate1, gate2 rows and biases
            inp["weights"][s]["mod_w"][chunk * D:(chunk + 1) * D] = 0
            inp["weights"][s]["mod_b"][chunk * D:(chunk + 1) * D] = 0
    gi, gt, _ = run_block(d, cfg, inp)
    np.testing.assert_array_equal(gi, si.as_f64(inp["x_img"], "bf16"))
    np.testing.assert_array_equal(gt, si.as_f64(inp["x_txt"], "bf16"))


def test_block_deterministic(d):
    cfg = si.CONFIGS["small_bf16"]
    inp = si.block_inputs(cfg)
    a = run_block(d, cfg, inp)
    b = run_block(d, cfg, inp)
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])


def test_block_mlp_half(d):
    cfg = si.CONFIGS["small_bf16"]
    inp = si.block_inputs(cfg)
    gi, gt, _ = run_block(d, cfg, inp, mlp_only=True)
    w64 = weights_f64(inp["weights"], cfg.dtype)
    temb = inp["temb"].astype(np.float64)
    for s, g, x in (("img", gi, inp["x_img"]), ("txt", gt, inp["x_txt"])):
        x64 = si.as_f64(x, cfg.dtype)
        for b in range(cfg.batch):
            m = {k: v[0] for k, v in O.modulation(temb[b:b + 1], w64[s]["mod_w"], w64[s]["mod_b"]).items()}
            check(cfg, g[b], O.mlp_half(w64[s], m, x64[b]), x64[b])


def test_block_mlp_long_k_ragged(d):
    """MLP half whose down projection has K >= 8192 on partial tiles (64 x 64 ones whose waves share K): 189 image
    and 63 text rows, 2176 output columns; every row is compared."""
    cfg = si.CONFIGS["mlp_long_k"]
    assert cfg.mlp_hidden >= 8192 and cfg.hidden % 256 != 0
    inp = si.block_inputs(cfg)
    gi, gt, _ = run_block(d, cfg, inp, mlp_only=True)
    w64 = weights_f64(inp["weights"], cfg.dtype)
    temb = inp["temb"].astype(np.float64)
    for s, g, x in (("img", gi, inp["x_img"]), ("txt", gt, inp["x_txt"])):
        x64 = si.as_f64(x, cfg.dtype)
        for b in range(cfg.batch):
            m = {k: v[0] for k, v in O.modulation(temb[b:b + 1], w64[s]["mod_w"], w64[s]["mod_b"]).items()}
            check(cfg, g[b], O.mlp_half(w64[s], m, x64[b]), x64[b])


@pytest.mark.parametrize("name", ["mlp_short_k128", "mlp_short_k192"])
def test_block_mlp_short_k_large_tiles(d, name):
    """MLP half whose up projection has only two or three k-tiles (K = 128, 192) on enough rows
    (16 x 4196) for the 256 x 256 tile path, the text stream's 1600 rows ending in a partial row
    tile: sampled rows of both streams against the oracle."""
    cfg = si.CONFIGS[name]
    inp = si.block_inputs(cfg)
    gi, gt, _ = run_block(d, cfg, inp, mlp_only=True)
    w64 = weights_f64(inp["weights"], cfg.dtype)
    rng = np.random.default_rng(11)
    for b in (0, cfg.batch - 1):
        for s, g, x, n in (("img", gi, inp["x_img"], cfg.n_img), ("txt", gt, inp["x_txt"], cfg.n_txt)):
            mm = O.modulation(inp["temb"][b:b + 1].astype(np.float64), w64[s]["mod_w"], w64[s]["mod_b"])
            m = {k: v[0] for k, v in mm.items()}
            rows = np.unique(np.r_[0, n - 1, rng.choice(n, 40, replace=False)])
            x64 = si.as_f64(x[b], cfg.dtype)[rows]
            check(cfg, g[b][rows], O.mlp_half(w64[s], m, x64), x64)


def test_block_concurrent_host_threads_on_two_streams(d):
    """Two host threads, each with its own stream, workspace and inputs, run block stacks at the same
    time (different weights and seeds, one of them at the 256 x 256 tile path's size); each result
    must equal, bit for bit, the same calls made one after the other."""
    import threading
    cfgs = [si.CONFIGS["small_bf16"], si.CONFIGS["mlp_short_k128"]]
    inps = [si.block_inputs(c, seed=si.MASTER_SEED + 1 + i) for i, c in enumerate(cfgs)]

    def prepare(cfg, inp):
        c = block_cfg(d, cfg)
        w = upload_block(inp["weights"], cfg.dtype)
        return (c, d.block_weights(w["img"], w["txt"]), dev(inp["temb"]), dev(inp["x_img"], cfg.dtype),
                dev(inp["x_txt"], cfg.dtype), d.workspace(d.dit_block_workspace_bytes(c, cfg.batch)), w)

    def run(args, stream, reps):
        c, bw, temb, xi, xt, ws, _ = args
        with torch.cuda.stream(stream):
            for _ in range(reps):
                d.dit_block_forward(c, bw, temb, xi, xt, ws, stream=stream)
        stream.synchronize()

    reps = 3
    seq = [prepare(c, i) for c, i in zip(cfgs, inps)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for a, st in zip(seq, streams):
        run(a, st, reps)
    par = [prepare(c, i) for c, i in zip(cfgs, inps)]
    errs = []

    def worker(a, st):
        try:
            run(a, st, reps)
        except Exception as e:   # reported after the join
            errs.append(e)
    threads = [threading.Thread(target=worker, args=(a, st)) for a, st in zip(par, streams)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errs, errs
    for a, b in zip(seq, par):
        assert torch.equal(a[3], b[3]) and torch.equal(a[4], b[4])


def test_block_errors_write_nothing(d):
    cfg = si.CONFIGS["small_bf16"]
    inp = si.block_inputs(cfg)
    c = block_cfg(d, cfg)
    w = upload_block(inp["weights"], cfg.dtype)
    bw = d.block_weights(w["img"], w["txt"])
    temb, xi, xt = dev(inp["temb"]), dev(inp["x_img"], "bf16"), dev(inp["x_txt"], "bf16")
    before = xi.clone()
    need = d.dit_block_workspace_bytes(c, cfg.batch)
    with pytest.raises(d.DitError) as ei:
        d.dit_block_forward(c, bw, temb, xi, xt, d.workspace(need - 256))
    assert ei.value.name == "DIT_ERR_WORKSPACE"
    bad = d.block_config(cfg.hidden, cfg.heads, cfg.head_dim, cfg.mlp_hidden, cfg.n_img + 1, cfg.n_txt,
                         cfg.grid_h, cfg.grid_w)                     # n_img != grid_h * grid_w
    with pytest.raises(d.DitError) as ei:
        d.dit_block_forward(bad, bw, temb, xi, xt, d.workspace(need))
    assert ei.value.name == "DIT_ERR_SHAPE"
    torch.cuda.synchronize()
    assert torch.equal(xi, before)


def _sampled(cfg, inp, gi, gt, batches, n_rows=24):
    w64 = weights_f64(inp["weights"], cfg.dtype)
    rng = np.random.default_rng(7)
    for b in batches:
        ir = np.unique(np.r_[0, cfg.n_img - 1, rng.choice(cfg.n_img, n_rows, replace=False)])
        tr = np.unique(np.r_[0, cfg.n_txt - 1, rng.choice(cfg.n_txt, n_rows // 3, replace=False)])
        xi = si.as_f64(inp["x_img"][b], cfg.dtype)
        xt = si.as_f64(inp["x_txt"][b], cfg.dtype)
        ri, rt = O.block_forward_sample(cfg, w64, inp["temb"][b].astype(np.float64), xi, xt, ir, tr)
        check(cfg, gi[b][ir], ri, xi[ir])
        check(cfg, gt[b][tr], rt, xt[tr])


@pytest.mark.parametrize("name", ["block_512", "block_1280"])
def test_block_full_size_sampled(d, name):
    cfg = si.CONFIGS[name]
    inp = si.block_inputs(cfg)
    gi, gt, _ = run_block(d, cfg, inp)
    assert np.all(np.isfinite(gi)) and np.all(np.isfinite(gt))
    _sampled(cfg, inp, gi, gt, [0, cfg.batch - 1])


def test_block_step_shape_sampled(d):
    """One block at the full-step launch shape (K=16, 1024 + 256 tokens)."""
    cfg = dataclasses.replace(si.CONFIGS["step_512_k16"], blocks=1)
    inp = si.block_inputs(cfg)
    gi, gt, _ = run_block(d, cfg, inp)
    _sampled(cfg, inp, gi, gt, [5])


def test_mlp_slice_full_size_sampled(d):
    """The per-token MLP half on one sequence-parallel rank's 1600 + 128 token slice."""
    cfg = si.CONFIGS["mlp_slice_1280"]
    inp = si.block_inputs(cfg)
    gi, gt, _ = run_block(d, cfg, inp, mlp_only=True)
    w64 = weights_f64(inp["weights"], cfg.dtype)
    rng = np.random.default_rng(3)
    for b in (0, cfg.batch - 1):
        m = {}
        for s in ("img", "txt"):
            mm = O.modulation(inp["temb"][b:b + 1].astype(np.float64), w64[s]["mod_w"], w64[s]["mod_b"])
            m[s] = {k: v[0] for k, v in mm.items()}
        ir = rng.choice(cfg.n_img, 32, replace=False)
        xi = si.as_f64(inp["x_img"][b], cfg.dtype)
        check(cfg, gi[b][ir], O.mlp_half(w64["img"], m["img"], xi[ir]), xi[ir])
        xt = si.as_f64(inp["x_txt"][b], cfg.dtype)
        check(cfg, gt[b], O.mlp_half(w64["txt"], m["txt"], xt), xt)
