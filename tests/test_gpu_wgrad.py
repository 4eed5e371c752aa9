"""The weight gradients' grouped product at the edges of its tiles and chunks:
token counts around 64, 256 and the change from 128- to 256-wide tiles, ragged
widths, every mode, against the oracle with the gates of the other parity tests;
and their sums bit for bit the same whichever stream and workspace content."""
import pytest
import torch

import paper_2605_03667_amd as elas
from oracle import ffn as offn
from synthetic import ffn_inputs
from tests.helpers import dev_bf16
from tests.test_gpu_ffn import compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["sparse", "dense", "ste"])
@pytest.mark.parametrize("T,d,F,r", [(63, 264, 520, 136), (65, 8, 8, 8), (193, 256, 256, 256), (4161, 600, 1096, 264),
                                     (12289, 1024, 1288, 256)])
def test_wgrad_edges(T, d, F, r, mode):
    bits = ffn_inputs(T, d, F, r, seed_base=T + F)
    f, b = offn.run(bits, sparse=(mode != "dense"), ste=(mode == "ste"))
    compare(run_gpu(bits, mode=mode), f, b, bits, mode=mode)


def test_wgrad_ignores_workspace_content():
    T, d, F, r = 4161, 600, 1096, 264
    t = {k: dev_bf16(v) for k, v in ffn_inputs(T, d, F, r, seed_base=3).items()}
    w = [t[k] for k in ("U_up", "V_up", "U_down", "V_down")]
    saved = elas.elas_lowrank_ffn_fwd(t["x"], *w)
    n = elas.elas_lowrank_ffn_bwd_workspace_bytes(T, d, F, r)
    ref = None
    for fill in (0, 255):
        ws = torch.full((n,), fill, dtype=torch.uint8, device="cuda:0")
        g = elas.elas_lowrank_ffn_bwd(t["dY"], t["x"], *w, saved, workspace=ws)
        if ref is not None:
            for k in g:
                assert torch.equal(g[k], ref[k]), k
        ref = g
