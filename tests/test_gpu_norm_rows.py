"""The norm of many rows (a row per wave) against the norm of few (a row per workgroup), launched by themselves: the same bits."""
import ctypes as C
import pytest
from test_gpu_products import _lib, _ptr

pytestmark = pytest.mark.gpu


def _norm(arch, h, g, b, out):
    """Normalises the rows of h into operand tiles `out`, in one launch."""
    import torch
    n = torch.tensor([h.shape[0]], dtype=torch.int32, device="cuda")
    _lib()["_ZN8sprinter11launch_normEiiPKfS1_S1_fiPKiPvPfiP12ihipStream_tPKNS_11NormPendingEPKNS_11EmbedSourceE"](
        1, arch, _ptr(h), _ptr(g), _ptr(b), C.c_float(1e-5), h.shape[1], _ptr(n), _ptr(out), _ptr(None), h.shape[0],
        C.c_void_p(torch.cuda.current_stream().cuda_stream), _ptr(None), _ptr(None))
    torch.cuda.synchronize()


# both sides of the rule's lines; columns that leave a k tile a quarter full, a chunk's lanes idle, and fill 1, 2 and 4 blocks of 2048
@pytest.mark.parametrize("arch", [0, 1])
@pytest.mark.parametrize("rows,d", [(3072, 8), (3073, 200), (3100, 1600), (1536, 2048), (1539, 2056), (1602, 4096), (1537, 8192)])
def test_row_per_wave_matches_row_per_workgroup(arch, rows, d):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + d)
    h = torch.randn(rows, d, device="cuda", generator=g) * 3 + 0.5
    gain, off = 1 + 0.1 * torch.randn(d, device="cuda", generator=g), 0.1 * torch.randn(d, device="cuda", generator=g)
    Kt, tiles = -(-d // 32), -(-rows // 16)
    whole, parts = (torch.full((tiles, Kt, 512), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    _norm(arch, h, gain, off, whole)
    for at in range(0, rows, 1024):                            # (a multiple of a row tile, below every line of the rule)
        _norm(arch, h[at:at + 1024].contiguous(), gain, off, parts[at // 16:])
    assert torch.equal(whole.view(torch.int16), parts.view(torch.int16))
    written = parts.view(tiles, Kt, 4, 16, 8).permute(0, 3, 1, 2, 4).reshape(tiles * 16, Kt * 32)
    assert not written[:rows, :d].isnan().any() and written[rows:].isnan().all() and written[:, d:].isnan().all()
