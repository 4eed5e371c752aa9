"""The weight gradients' grouped product at the edges of its tiles and chunks:
token counts around 64, 256 and the change from 128- to 256-wide tiles, ragged
widths, every mode, against the oracle with the gates of the other parity tests;
with inputs whose every sum is exact in binary32, against the oracle bit for bit,
so that no token of any chunk or ragged end may be missing; and their sums bit for
bit the same whichever stream and workspace content."""
import numpy as np
import pytest
import torch

import paper_2605_03667_amd as elas
from oracle import ffn as offn
from synthetic import ffn_inputs
from tests.helpers import dev_bf16
from tests.test_gpu_ffn import GRADS, all_sums_exact, compare, run_gpu, sparse_sign_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["sparse", "dense", "ste"])
@pytest.mark.parametrize("T,d,F,r", [(63, 264, 520, 136), (65, 8, 8, 8), (193, 256, 256, 256), (4161, 600, 1096, 264),
                                     (12289, 1024, 1288, 256)])
def test_wgrad_edges(T, d, F, r, mode):
    bits = ffn_inputs(T, d, F, r, seed_base=T + F)
    f, b = offn.run(bits, sparse=(mode != "dense"), ste=(mode == "ste"))
    compare(run_gpu(bits, mode=mode), f, b, bits, mode=mode)


# 128-wide tiles in 3 chunks; 256-wide ones in 8 chunks whose last step holds 1 token of
# a new block of 256, 63 tokens, and 1 token of a block's last step
@pytest.mark.parametrize("mode", ["sparse", "dense", "ste"])
@pytest.mark.parametrize("T,d,F,r", [(705, 264, 520, 136), (4097, 600, 1096, 264), (4159, 600, 1096, 264),
                                     (4289, 600, 1096, 264)])
def test_wgrad_exact(T, d, F, r, mode):
    bits = sparse_sign_inputs(T, d, F, r, [1 / 16, 1 / 16, 1 / 32, 1 / 8, 1 / 8, 1 / 4], [0, 0, 0, -8, -4, 0], 51)
    f, b = offn.run(bits, sparse=(mode != "dense"), ste=(mode == "ste"))
    assert all_sums_exact(bits, f, b)
    for name, v in (("x", bits["x"]), ("P", f["P"]), ("S", f["S"]), ("Z", f["Z"]), ("dY", bits["dY"]), ("dZ", b["dZ"]),
                    ("dH", b["dH"]), ("dP", b["dP"])):
        assert np.all(np.any((v & 0x7FFF if v.dtype == np.uint16 else v) != 0, axis=1)), name   # every token contributes
    gpu = run_gpu(bits, mode=mode)
    for k in GRADS:
        np.testing.assert_array_equal(gpu[k], b[k], err_msg=k)


def test_wgrad_ignores_stream_and_workspace_content():
    T, d, F, r = 4161, 600, 1096, 264
    t = {k: dev_bf16(v) for k, v in ffn_inputs(T, d, F, r, seed_base=3).items()}
    w = [t[k] for k in ("U_up", "V_up", "U_down", "V_down")]
    saved = elas.elas_lowrank_ffn_fwd(t["x"], *w)
    n = elas.elas_lowrank_ffn_bwd_workspace_bytes(T, d, F, r)
    ref = None
    for fill, stream in ((0, None), (255, None), (127, torch.cuda.Stream())):
        ws = torch.full((n,), fill, dtype=torch.uint8, device="cuda:0")
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            g = elas.elas_lowrank_ffn_bwd(t["dY"], t["x"], *w, saved, workspace=ws)
        torch.cuda.synchronize()
        if ref is not None:
            for k in g:
                assert torch.equal(g[k], ref[k]), k
        ref = g
