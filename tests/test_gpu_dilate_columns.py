"""Dilation of a mask with more than 2^32 columns of words, which a thread per
column cannot cover in one launch: set voxels in the first and the last frame, all
other words stay zero."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_more_columns_than_threads_of_a_launch():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    dims = (64, 65540, 2, 65535)  # 65535 x 65540 columns of one word and two slices
    assert dims[1] * dims[3] > 1 << 32
    n = dims[1] * dims[2] * dims[3]
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (2 * 8 * n + (8 << 30)):
        pytest.skip("needs 150 GB of device memory")
    a, b = torch.zeros(n, dtype=torch.int64, device="cuda"), torch.full((n,), -1, device="cuda")
    at = lambda t, z, y: (t * dims[2] + z) * dims[1] + y  # noqa: E731
    a[at(0, 0, 5)] = 1 << 20
    a[at(dims[3] - 1, 1, dims[1] - 1)] = 1
    p = C.c_void_p
    fl._check(fl.lib().fhash_dilate_mask(p(a.data_ptr()), (C.c_int64 * 4)(*dims), C.c_int32(1),
                                         p(b.data_ptr()),
                                         p(torch.cuda.current_stream().cuda_stream)), "dilate")
    want = {at(0, z, y): 7 << 19 for z in (0, 1) for y in (4, 5, 6)}
    want.update({at(dims[3] - 1, z, y): 3 for z in (0, 1) for y in (dims[1] - 2, dims[1] - 1)})
    got = {}
    for i in range(0, n, 1 << 29):
        part = b[i:i + (1 << 29)]
        for k in part.nonzero().flatten().tolist():
            got[i + k] = part[k].item()
    del a, b
    torch.cuda.empty_cache()
    assert got == want
