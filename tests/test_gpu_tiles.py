"""Edges of the tiled bf16 contraction (photon_chunker_project, Eq. 4) against an fp32 product of the same bf16 inputs."""
import pytest
import torch

from util import require_gpu

pytestmark = pytest.mark.gpu


# 192 tiles of 256 x 256 and up: the counter-phase kernel.  One row more and one less than whole row tiles, a last
# column tile of 16 columns, one to three K slabs, a tile count that is no multiple of 8.
@pytest.mark.parametrize("rows,K,N", [(6144, 64, 2048), (6145, 128, 2048), (6143, 192, 2048), (49409, 64, 256), (6100, 320, 2064)])
def test_tiled_contraction_edges(rows, K, N):
    require_gpu()
    import paper_2512_20687_amd as ph
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    x = torch.randn((rows, K), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.1).to(torch.bfloat16)
    b = torch.randn((N,), generator=g, device="cuda")
    out = torch.full((rows + 1, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ph.photon_chunker_project(x, w, b, out[:rows], 1)
    torch.cuda.synchronize()
    assert bool(torch.isnan(out[rows]).all())                       # nothing is stored past the last row
    ref = x.float() @ w.float().t() + b
    # one rounding of the output to bf16 (2^-9 of its value) and fp32 sums of K products in two orders
    err = (out[:rows].float() - ref).abs()
    bound = ref.abs() * 2.0 ** -8 + 1e-5 * K ** 0.5
    assert bool((err <= bound).all()), float((err - bound).max())
