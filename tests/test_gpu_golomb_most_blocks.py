"""PivCo-Golomb encode at the most blocks that one launch covers with a workgroup
of 256 threads each (2^24 - 1, a grid of fewer than 2^32 threads), and one more,
which is refused before anything is launched."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2606_05765_amd.pivco")

MOST = (1 << 24) - 1


def test_limit():
    room = int(P.lib().pivco_golomb_encode_workspace(MOST + 1, 1))
    if torch.cuda.mem_get_info()[0] < room + (4 << 30):
        pytest.skip("needs 73 GB of device memory")
    ws = torch.empty(room, dtype=torch.uint8, device="cuda")
    for n, rc in ((MOST, P.OK), (MOST + 1, P.E_DEVICE)):
        print("blocks", n, flush=True)
        x = torch.zeros(n, dtype=torch.uint8, device="cuda")
        size = 32 + 8 * (n + 1) + 16 * n       # a block: 12 bytes of header, one bit, padding
        out = torch.full((size + 64,), 0xAB, dtype=torch.uint8, device="cuda")
        length = C.c_uint64(0)
        got = P.lib().pivco_golomb_encode(x.data_ptr(), n, 1, out.data_ptr(), size, C.byref(length), ws.data_ptr(),
                                          room, C.c_void_p(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        assert got == rc
        if rc != P.OK:
            assert (out == 0xAB).all()
            continue
        assert length.value == size and (out[size:] == 0xAB).all()
        w = out[:size].view(torch.int32)
        assert w[4].item() == 1 and w[5].item() == n
        tab = out[32:32 + 8 * (n + 1)].view(torch.int64)
        assert (tab == 32 + 8 * (n + 1) + 16 * torch.arange(n + 1, device="cuda")).all()
        blocks = out[32 + 8 * (n + 1):size].view(torch.int32).view(n, 4)
        assert (blocks == torch.tensor([13, 1, 1, 1], dtype=torch.int32, device="cuda")).all()
    del ws
    torch.cuda.empty_cache()
