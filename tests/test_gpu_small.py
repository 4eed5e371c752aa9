"""The wave-split products at the edges of their blocks: token counts around 16,
32 and 64, contractions that are no multiple of 64 or of the waves' chunks, and
feature counts that are no multiple of 16 or 64, against the oracle with the
gates of the other parity tests; the orientation of the factors, which decides
between them, the token-resident and the tiled kernel, must not show in any
output; and neither must the kernel that a token count selects: the sums over K
are cut and ordered as in the tiled kernels, whose recorded outputs the
wave-split ones (one case or more for each of their shapes) match bit for bit."""
import hashlib
import os

import pytest
import torch

import paper_2605_03667_amd as elas
from oracle import ffn as offn
from synthetic import ffn_inputs
from tests.helpers import dev_bf16
from tests.test_gpu_ffn import compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["sparse", "dense", "ste"])
@pytest.mark.parametrize("T,d,F,r", [(16, 2056, 72, 512), (17, 520, 5464, 520), (48, 2048, 200, 256),
                                     (250, 1032, 1000, 264), (1023, 776, 328, 128)])
def test_small_edges(T, d, F, r, mode):
    bits = ffn_inputs(T, d, F, r, seed_base=T + d)
    f, b = offn.run(bits, sparse=(mode != "dense"), ste=(mode == "ste"))
    compare(run_gpu(bits, mode=mode), f, b, bits, mode=mode)


@pytest.mark.parametrize("T,d,F,r", [(1, 2048, 5464, 512), (100, 768, 2048, 256), (500, 1024, 2736, 256),
                                     (1100, 512, 1376, 128), (2000, 2048, 5464, 512)])
def test_factor_orientation_identical(T, d, F, r):
    t = {k: dev_bf16(v) for k, v in ffn_inputs(T, d, F, r, seed_base=6).items()}
    w = [t[k] for k in ("U_up", "V_up", "U_down", "V_down")]
    a = elas.elas_lowrank_ffn_fwd(t["x"], *w)
    b = elas.elas_lowrank_ffn_fwd(t["x"], *[x.t().contiguous() for x in w], flags=elas.ELAS_FACTORS_AB)
    for k in a:
        assert torch.equal(a[k], b[k]), k


def _recorded():
    with open(os.path.join(os.path.dirname(__file__), "golden", "few_token_bits.txt")) as f:
        for line in f:
            if not line.startswith("#"):
                T, d, F, r, mode, *bits = line.split()
                yield pytest.param(int(T), int(d), int(F), int(r), mode, bits, id=f"{T}-{d}-{F}-{r}-{mode}")


@pytest.mark.parametrize("T,d,F,r,mode,bits", _recorded())
def test_outputs_are_the_tiled_kernels(T, d, F, r, mode, bits):
    t = {k: dev_bf16(v) for k, v in ffn_inputs(T, d, F, r, seed_base=T + r).items()}
    w = [t[k] for k in ("U_up", "V_up", "U_down", "V_down")]
    flags = elas.ELAS_MODE_DENSE if mode == "dense" else 0
    o = elas.elas_lowrank_ffn_fwd(t["x"], *w, flags=flags)
    g = elas.elas_lowrank_ffn_bwd(t["dY"], t["x"], *w, o, flags=elas.ELAS_BWD_STE if mode == "ste" else flags)
    got = [hashlib.sha1(a.view(torch.int16).cpu().numpy().tobytes()).hexdigest()[:12] for a in (o["P"], o["Z"], o["y"], g["dx"])]
    assert dict(zip(("P", "Z", "y", "dx"), got)) == dict(zip(("P", "Z", "y", "dx"), bits))
