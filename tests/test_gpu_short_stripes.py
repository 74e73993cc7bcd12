"""GPU: whole-path renders of sets whose tensors are all shorter than one stripe.

The wave renders such a tensor piece by piece up to 16 chunks and a chunk per lane
beyond: lengths of one row, around 8 KiB (what it holds in flight) and around 16
chunks, for every row size that takes this variant (64, 128 and 256 bytes), both
pairings, one head and several (the merged rows of two heads are not adjacent), with
a re-delivered fragment, whose Id is known before the render."""

import pytest
import torch

import synth
import paper_2607_01308_amd as cm
from gpu_util import check_render, gpu_deliveries

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("style", ["half", "interleaved"])
@pytest.mark.parametrize("H", [1, 3])
@pytest.mark.parametrize("dtype,d", [("bfloat16", 32), ("bfloat16", 64), ("float32", 16),
                                     ("float32", 64), ("bfloat16", 128)])
def test_short_stripe_edges(dtype, d, H, style):
    row = H * d * (4 if dtype == "float32" else 2)
    half, limit = 8192 // row, 16384 // row
    w = synth.custom("short-edges", dtype=dtype, d=d, H=H, L=1, routing_layer=0,
                     lengths=(1, half, half + 1, limit, limit + 1),
                     deliveries=(0, 1, 2, 3, 4, 3), seed=d + H)
    _, dl = gpu_deliveries(w)
    res = cm.render_deliveries(dl, 0, w.rope_base, style=style)
    torch.cuda.synchronize()
    check_render(res, dl, w.dtype, 0, w.rope_base, style=style)
