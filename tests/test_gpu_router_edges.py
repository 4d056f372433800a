"""The router at the edges of its workspace and of its tile rule, bit for bit
against the oracle's ordered fp32 sums."""

import numpy as np
import pytest
import torch

import oracle
from paper_2511_11505_amd import _lib as L
from tests._util import f64
from workloads import CONFIGS

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]
DEV = "cuda"
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


def route(dtype, N, d, E):
    """Logits of a router of E experts over N tokens; the workspace is the
    stated size to the byte, and 1 KiB behind it has to stay as it was."""
    desc = L.make_desc(CONFIGS["tiny"].scaled(n_tokens=N, hidden=d, n_experts=E, top_k=2, dtype=dtype))
    gen = torch.Generator(device=DEV).manual_seed(N + d + E)
    x = torch.randn((N, d), generator=gen, device=DEV).to(TORCH[dtype])
    w = (0.05 * torch.randn((E, d), generator=gen, device=DEV)).to(TORCH[dtype])
    logits = torch.empty((N, E), dtype=torch.float32, device=DEV)
    ids = torch.empty((N, 2), dtype=torch.int32, device=DEV)
    tw = torch.empty((N, 2), dtype=torch.float32, device=DEV)
    nbytes = L.fs_workspace_size(desc, L.FS_OP_ROUTER_TOPK)
    ws = torch.full((nbytes + 1024,), 0xA5, dtype=torch.uint8, device=DEV)
    L.fs_router_topk(desc, x, w, None, None, logits, ids, tw, (ws.data_ptr(), nbytes))
    torch.cuda.synchronize()
    assert bool((ws[nbytes:] == 0xA5).all()), "wrote past the workspace"
    z = logits.cpu().numpy()
    ref = oracle.logits_routing_f32(f64(x).astype(np.float32), f64(w).astype(np.float32))
    assert np.array_equal(z, ref)


# slice sums whose size is not a multiple of 256 bytes, beside sizes that are
@pytest.mark.parametrize("dtype,N,d,E", [("f32", 1, 7168, 8), ("bf16", 1, 7168, 8),
                                         ("bf16", 129, 7168, 8), ("f32", 3, 1152, 60),
                                         ("bf16", 16, 2048, 64)])
def test_router_workspace_bound(dtype, N, d, E):
    route(dtype, N, d, E)
