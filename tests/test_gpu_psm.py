"""GPU parity of the Patch Selection Module forward pass (litevlm_psm_forward)
against the oracle's psm_forward.

The GPU rounds every GEMM and attention input to bf16 (fp32 accumulation), so
the logits carry a few parts in a thousand of the activations' scale; the bound
|got - ref| <= 2e-2 + 2e-2*|ref| leaves about 4x headroom over what the bf16
rounding of 4 layers gives. The view decisions of the patch selection made from
the GPU logits must equal the oracle's wherever a logit is not within 0.1 of the
threshold's logit (0 at w_lexical 0, threshold 0.5)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_07416_amd as lv
import synth
from oracle import psm as OP
from parity_util import log

pytestmark = pytest.mark.gpu

PSM_RTOL, PSM_ATOL = 2e-2, 2e-2

CASES = [
    ("2 layers, 16 tokens, d 256", dict(B=1, T=16, d=256, H=4, dff=512, N=6, L=2)),
    ("benchmark shape: 4 layers, 128 tokens, d 256, batch 3", dict(B=3, T=128, d=256, H=4, dff=1024, N=6, L=4)),
    ("d 512, head dim 128, ragged 37 tokens", dict(B=2, T=37, d=512, H=4, dff=256, N=3, L=1)),
]


def run(c, seed):
    emb, par = synth.psm_inputs(c["B"], c["T"], c["d"], c["dff"], c["N"], c["L"], seed)
    out = lv.psm_forward(torch.from_numpy(emb).cuda(), torch.from_numpy(par).cuda(), c["H"], c["dff"], c["N"], c["L"])
    torch.cuda.synchronize()
    ref = OP.psm_forward(emb.astype(np.float64), par.astype(np.float64), c["H"], c["dff"], c["N"], c["L"])
    return out, ref


@pytest.mark.parametrize("name,c", CASES)
def test_psm_matches_oracle(name, c):
    out, ref = run(c, seed=5100 + c["T"])
    got = out.cpu().numpy().astype(np.float64)
    err = np.abs(got - ref)
    assert np.all(err <= PSM_ATOL + PSM_RTOL * np.abs(ref)), f"{name}: max err {err.max():.3g}"
    log(f"{name}: logits max abs err {err.max():.2e} (|ref| max {np.abs(ref).max():.2f})")
    # the patch selection made from these logits
    vk, _, _ = lv.patch_select(out, np.arange(c["N"] + 1) * 4, 4 * c["N"] + 1, 0.0, 0.5)
    vk_ref = oracle.patch_select(ref.astype(np.float32), None, 0.0, 0.5)
    clear = np.abs(ref) > 0.1
    assert np.array_equal(vk.cpu().numpy()[clear], vk_ref[clear])


def test_psm_is_deterministic():
    c = CASES[1][1]
    a, _ = run(c, seed=5200)
    b, _ = run(c, seed=5200)
    assert torch.equal(a, b)


# Where the tiles, chunks and folds end: one token; rows past a 32-row tile; k
# ranges shorter than a chunk and cut short in the last one; more views than a
# pass of the fold takes, an odd number of them; each tile size of the GEMMs (64
# x 64 from 192 tiles on, 64 x 128 from 512) with a last row tile cut short.
EDGES = [
    ("one token, one view", dict(B=1, T=1, d=256, H=4, dff=64, N=1, L=1)),
    ("65 rows, d_ff 320", dict(B=1, T=65, d=256, H=2, dff=320, N=9, L=2)),
    ("64 views, d 512, d_ff 576", dict(B=3, T=33, d=512, H=8, dff=576, N=64, L=1)),
    ("64 x 64 tiles, 1010 rows", dict(B=5, T=202, d=256, H=4, dff=1024, N=5, L=2)),
    ("64 x 64 tiles, d 512, 1450 rows", dict(B=2, T=725, d=512, H=4, dff=1088, N=3, L=1)),
    ("64 x 128 tiles, d 512, 2060 rows", dict(B=4, T=515, d=512, H=8, dff=2048, N=6, L=1)),
    ("64 x 128 tiles, d 256, 5500 rows", dict(B=20, T=275, d=256, H=4, dff=1024, N=6, L=1)),
    # the residual GEMMs (bf16 rows in) reach 64 x 128 from 8129 rows at d 512
    ("64 x 128 tiles in the residual GEMMs too, 8150 rows", dict(B=50, T=163, d=512, H=8, dff=576, N=6, L=1)),
]


@pytest.mark.parametrize("name,c", EDGES)
def test_psm_edges(name, c):
    out, ref = run(c, seed=5300 + c["T"])
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
    # the bound of the shapes above: bf16 GEMM inputs over at most two layers
    assert np.all(err <= PSM_ATOL + PSM_RTOL * np.abs(ref)), f"{name}: max err {err.max():.3g}"
    log(f"{name}: logits max abs err {err.max():.2e} (|ref| max {np.abs(ref).max():.2f})")


def param(par, c, name):
    """The named part of the flat parameter vector (a view)."""
    off = 0
    for nm, shape in OP.param_layout(c["d"], c["dff"], c["N"], c["L"]):
        n = int(np.prod(shape))
        if nm == name:
            return par[off:off + n].reshape(shape)
        off += n
    raise KeyError(name)


@pytest.mark.parametrize("d", [256, 512])
def test_psm_cross_logits_at_minus_infinity(d):
    """Tokens whose cross-attention logit leaves the range of fp32 downwards have
    no weight, wherever they stand among the others."""
    c = dict(B=1, T=40, d=d, H=4, dff=64, N=3, L=1)
    emb, par = synth.psm_inputs(c["B"], c["T"], d, c["dff"], c["N"], c["L"], seed=5400)
    for n in ("l0.w_o", "l0.b_o", "l0.w_down", "l0.b_down", "latents", "b_ck", "lnf_b"):
        param(par, c, n)[:] = 0.0  # the encoder passes the embeddings on
    # the final norm leaves rows of +-1 as they are; logits of -1e38 * d or (rows orthogonal to p) 0
    i = np.arange(d)
    p, r = np.where(i % 2 == 0, 1.0, -1.0), np.where(i % 4 < 2, 1.0, -1.0)
    param(par, c, "lnf_g")[:] = 1.0
    param(par, c, "b_cq")[:] = 1e30 * p
    param(par, c, "w_ck")[:] = 1e8 * np.eye(d)
    emb[0] = r
    emb[0, 3:30:4] = -r
    emb[0, [0, 7, 33]] = -p
    out = lv.psm_forward(torch.from_numpy(emb).cuda(), torch.from_numpy(par).cuda(), c["H"], c["dff"], c["N"], c["L"])
    torch.cuda.synchronize()
    ref = OP.psm_forward(emb.astype(np.float64), par.astype(np.float64), c["H"], c["dff"], c["N"], c["L"])
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= PSM_ATOL + PSM_RTOL * np.abs(ref)), f"got {out.tolist()}, reference {ref.tolist()}"


@pytest.mark.parametrize("d", [256, 512])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_psm_parameters_that_are_no_numbers_show(d, value):
    """A NaN or an infinity in any parameter leaves no finite logit where the
    oracle's is not (b_ck, whose finite values the softmax cancels, included)."""
    c = dict(B=2, T=20, d=d, H=4, dff=64, N=3, L=2)
    emb, par = synth.psm_inputs(c["B"], c["T"], d, c["dff"], c["N"], c["L"], seed=5500)
    for name, _ in OP.param_layout(d, c["dff"], c["N"], c["L"]):
        x = par.copy()
        a = param(x, c, name).reshape(-1)
        a[a.size // 2] = value
        out = lv.psm_forward(torch.from_numpy(emb).cuda(), torch.from_numpy(x).cuda(), c["H"], c["dff"], c["N"], c["L"])
        torch.cuda.synchronize()
        with np.errstate(all="ignore"):
            ref = OP.psm_forward(emb.astype(np.float64), x.astype(np.float64), c["H"], c["dff"], c["N"], c["L"])
        assert np.array_equal(np.isfinite(out.cpu().numpy()), np.isfinite(ref)), f"{name}: {out.tolist()}, reference {ref.tolist()}"
