"""What the library keeps resident on a GPU: the scratch array of sla2_router_static as sla2.h states it, and code."""
import struct

import pytest

from paper_2602_12675_amd import api

SCRATCH = 32 << 20                       # SLA2_STATIC_SCRATCH_BYTES
EM_AMDGPU, PT_LOAD = 224, 1


def _device_images(blob):
    """(offset, program headers) of every AMDGPU ELF image embedded in the library."""
    at = blob.find(b"\x7fELF", 1)
    while at >= 0:
        if len(blob) - at >= 64 and struct.unpack_from("<H", blob, at + 18)[0] == EM_AMDGPU:
            phoff, = struct.unpack_from("<Q", blob, at + 32)
            size, count = struct.unpack_from("<HH", blob, at + 54)
            yield [struct.unpack_from("<IIQQQQQQ", blob, at + phoff + n * size) for n in range(count)]
        at = blob.find(b"\x7fELF", at + 1)


def test_resident_size_is_one_scratch_array():
    with open(api.LIB_PATH, "rb") as f:
        blob = f.read()
    loads = [sum(h[6] for h in headers if h[0] == PT_LOAD) for headers in _device_images(blob)]     # p_memsz
    assert loads, "no device image found"
    assert max(loads) >= SCRATCH                               # the array is where this test looks for it
    assert sum(loads) <= SCRATCH + (4 << 20)                   # the code of all kernels is below 2 MiB


@pytest.mark.gpu
def test_static_router_at_the_limit_of_its_scratch():
    """18 heads of 75,600 tokens at d = 128 take 97 % of the array, and what fills it is read back right; 19 are refused."""
    import torch
    d, N, bq = 128, 75600, 128
    for H, fits in ((18, True), (19, False)):
        p = api.make_params(1, H, N, d, bq, 64, 0.02)
        need = api.sla2_workspace_layout(p).block_idx
        assert (need <= SCRATCH) == fits
        if not fits:
            assert api.sla2_router_static(p, 256, 256, 256, 256, check=False) == api.SLA2_EWORKSPACE
            continue
        assert need > 0.95 * SCRATCH
        g = torch.Generator(device="cuda").manual_seed(3)
        q, k = (torch.randn((1, H, N, d), generator=g, device="cuda").bfloat16() for _ in range(2))
        rw = torch.randn((2, d, d), generator=g, device="cuda") / d ** 0.5
        shape = (1, H, -(-N // bq), api.sla2_num_selected(p))
        want, got = (torch.full(shape, -1, dtype=torch.int32, device="cuda") for _ in range(2))
        api.sla2_router(p, q, k, rw, want, api.alloc_workspace(p))
        api.sla2_router_static(p, q, k, rw, got)
        assert torch.equal(want, got) and int(got.min()) >= 0
