"""The DITSTEP_DEBUG build (libditstep_debug.so: every launch synchronised and checked, every operand
range of the block path's GEMM, attention and LayerNorm launches checked against the buffers the
entry point knows) runs the block forward, the MLP-only entry and a denoise step without a finding,
and gives the same bits as the release build. Each library runs in a fresh process
(tests/debug_build_child.py)."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2606_19004_amd")


def _child(lib, path):
    env = dict(os.environ, DITSTEP_LIB=os.path.join(PKG, lib))
    r = subprocess.run([sys.executable, "-u", os.path.join(ROOT, "tests", "debug_build_child.py"), path],
                       capture_output=True, text=True, timeout=300, cwd=ROOT, env=env)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert r.stdout.strip().splitlines()[-1] == f"ok {lib}"
    return np.load(path)


def test_debug_build_runs_clean_and_matches_release(tmp_path):
    assert os.path.exists(os.path.join(PKG, "libditstep_debug.so")), "build() also builds the debug library"
    rel = _child("libditstep.so", str(tmp_path / "release.npz"))
    dbg = _child("libditstep_debug.so", str(tmp_path / "debug.npz"))
    assert sorted(rel.files) == sorted(dbg.files) and len(rel.files) == 10
    for k in rel.files:
        np.testing.assert_array_equal(dbg[k], rel[k], err_msg=k)


def test_debug_build_refuses_an_operand_outside_the_known_buffers():
    """With the workspace registered 4 KB short (a test hook of the debug build), the MLP-up GEMM's
    output reaches past it, and the launch is refused on the host with a debug-check error."""
    code = (
        "import sys; sys.path.insert(0, '.')\n"
        "import seeded_inputs as si, torch\n"
        "from tests.gpu_util import block_cfg, dev, upload_block\n"
        "from paper_2606_19004_amd import ditstep as d\n"
        "cfg = si.CONFIGS['small_bf16']; inp = si.block_inputs(cfg); c = block_cfg(d, cfg)\n"
        "w = upload_block(inp['weights'], cfg.dtype); bw = d.block_weights(w['img'], w['txt'])\n"
        "ws = d.workspace(d.dit_block_workspace_bytes(c, cfg.batch))\n"
        "try:\n"
        "    d.dit_block_mlp(c, bw, dev(inp['temb']), dev(inp['x_img'], cfg.dtype), dev(inp['x_txt'], cfg.dtype), ws)\n"
        "except d.DitError as e:\n"
        "    print('refused', e.name, str(e))\n"
        "else:\n"
        "    print('accepted')\n")
    env = dict(os.environ, DITSTEP_LIB=os.path.join(PKG, "libditstep_debug.so"), DITSTEP_DEBUG_SHRINK_WS="1")
    r = subprocess.run([sys.executable, "-u", "-c", code], capture_output=True, text=True, timeout=300, cwd=ROOT, env=env)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    last = r.stdout.strip().splitlines()[-1]
    assert last.startswith("refused DIT_ERR_INVALID_ARG") and "debug check: gemm_mlp_up_gelu" in last, last


def test_gated_step_waits_without_an_event():
    """Where no event can mark the distance's copy (a test hook of the debug build stands in for that), the gated step
    waits for its whole stream and decides and answers the same."""
    code = (
        "import sys; sys.path.insert(0, '.')\n"
        "import seeded_inputs as si, torch\n"
        "from tests.test_gpu_graph import gated_setup\n"
        "from paper_2606_19004_amd import ditstep as d\n"
        "step, st, bufs, lat0, keep = gated_setup(d, si.CONFIGS['small_step_bf16'])\n"
        "st.threshold = 0.3\n"
        "out = [step(0.8 - 0.05 * i, 0.75 - 0.05 * i) for i in range(8)]\n"
        "torch.cuda.synchronize()\n"
        "print(repr(out), bufs['lat'].double().sum().item(), bufs['v'].double().sum().item())\n")
    got = []
    for extra in ({}, {"DITSTEP_DEBUG_NO_EVENT": "1"}):
        env = dict(os.environ, DITSTEP_LIB=os.path.join(PKG, "libditstep_debug.so"), **extra)
        r = subprocess.run([sys.executable, "-u", "-c", code], capture_output=True, text=True, timeout=300, cwd=ROOT, env=env)
        assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
        got.append(r.stdout.strip().splitlines()[-1])
    assert got[0] == got[1] and "True" in got[0]
