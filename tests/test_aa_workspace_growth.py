"""The cached workspace of the one-shot calls, with layers that do store their rewritten operands in it (collected first, so that
the block starts small)."""
import numpy as np
import pytest
import torch

from oracle import direct
from paper_2104_04731_amd.inputs import CONFIGS

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_growth_keeps_captured_graphs_of_stored_layers_valid(lib):
    """A graph captured while the block was small replays right after a larger layer has moved the library to a bigger
    block (1.7 to 7.5 MB); a call that would have to grow it under capture (27 MB) is refused with nothing enqueued."""
    small, big, huge = CONFIGS["C4a"], CONFIGS["C4a"].scaled(96), CONFIGS["C4a"].scaled(400)
    for cfg in (small, big, huge):
        assert lib.query_stage(cfg.dims(), lib.ENTRY_ONE_SHOT)[0] == lib.STAGE_STORED
    x, w = small.make()
    want = direct.conv2d_int8(x, w, small.stride, small.pad)
    dx, dw = torch.from_numpy(x).to(DEV), torch.from_numpy(w).to(DEV)
    out = torch.empty(want.shape, dtype=torch.int32, device=DEV)
    lib.conv2d_int8(dx, dw, small.stride, small.pad, out=out)          # sizes the block
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        lib.conv2d_int8(dx, dw, small.stride, small.pad, out=out)
    gen = torch.Generator(device=DEV).manual_seed(4261)
    bx = torch.randint(-128, 128, (huge.N, huge.C, huge.H, huge.W), dtype=torch.int8, device=DEV, generator=gen)
    bout = lib.conv2d_int8(bx[:big.N], dw, big.stride, big.pad)        # grows it
    for n in (0, big.N - 1):
        assert np.array_equal(bout[n:n + 1].cpu().numpy(), direct.conv2d_int8(bx[n:n + 1].cpu().numpy(), w, 1, 1)), n
    for rep in range(3):
        out.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want), rep
        lib.conv2d_int8(bx[:big.N], dw, big.stride, big.pad, out=bout)
    hout = torch.full((huge.N, huge.K, huge.P, huge.Q), -7, dtype=torch.int32, device=DEV)
    g2 = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g2):
        lib.conv2d_int8(dx, dw, small.stride, small.pad, out=out)
        with pytest.raises(lib.ConvError) as e:
            lib.conv2d_int8(bx, dw, huge.stride, huge.pad, out=hout)
        assert e.value.status == lib.ERR_WORKSPACE
    for rep in range(3):
        out.fill_(-1)
        g2.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want) and int((hout[::97] != -7).sum()) == 0, rep
    lib.conv2d_int8(bx, dw, huge.stride, huge.pad, out=hout)
    n = huge.N - 1
    assert np.array_equal(hout[n:n + 1].cpu().numpy(), direct.conv2d_int8(bx[n:n + 1].cpu().numpy(), w, 1, 1))
