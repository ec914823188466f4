"""Values into the order of the transpose's entries: every entry moves exactly, whichever workgroups an XCD gets."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nnz", [1, 255, 257, 1793, 2048, 2049, 4000, 70001, 6000128, 6000129])
@pytest.mark.parametrize("elem_bytes", [2, 4])
def test_permute_values(nnz, elem_bytes):
    import torch
    import paper_2006_10901_amd as spdl
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9900 + nnz)
    perm = torch.randperm(nnz, generator=gen, device="cuda").to(torch.int32)
    dtype = torch.float16 if elem_bytes == 2 else torch.float32
    values = torch.randn(nnz, generator=gen, device="cuda").to(dtype)
    out = torch.full((nnz + 2,), float("nan"), device="cuda", dtype=dtype)
    spdl.spdl_permute_values(nnz, elem_bytes, perm, values, out[1:-1])
    torch.cuda.synchronize()
    assert torch.isnan(out[0]) and torch.isnan(out[-1])
    assert np.array_equal(out[1:-1].cpu().numpy(), values.cpu().numpy()[perm.cpu().numpy()])
