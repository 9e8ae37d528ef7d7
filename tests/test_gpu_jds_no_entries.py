"""CRS -> JDS of a row pointer without entries where the caller's count says
otherwise: there are no diagonals, jd_ptr holds one element and nothing past
it is looked at."""
import ctypes as C

import pytest
import torch

from paper_0910_4836_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 64, 300])
def test_count_without_entries(n):
    lib = _lib.load()
    dev = dict(dtype=torch.int32, device="cuda")
    row_ptr, col, perm, iperm = torch.zeros(n + 1, **dev), torch.zeros(5, **dev), torch.empty(n, **dev), torch.empty(n, **dev)
    val, jd_val = torch.ones(5, dtype=torch.float64, device="cuda"), torch.full((5,), 7.0, dtype=torch.float64, device="cuda")
    jd_ptr, jd_col = torch.full((1,), -1, **dev), torch.full((5,), -1, **dev)
    ws = torch.empty(lib.spmv_jds_from_csr_workspace_size(n, 5), dtype=torch.uint8, device="cuda")
    nd, h_ptr = C.c_int32(-1), (C.c_int32 * 1)(-1)
    _lib.call("spmv_jds_from_csr", n, 5, row_ptr.data_ptr(), col.data_ptr(), val.data_ptr(), _lib.F64, 0,
              perm.data_ptr(), iperm.data_ptr(), jd_ptr.data_ptr(), 1, jd_col.data_ptr(), jd_val.data_ptr(),
              C.byref(nd), h_ptr, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert nd.value == 0 and h_ptr[0] == 0 and jd_ptr.tolist() == [0]
    assert perm.tolist() == list(range(n)) and iperm.tolist() == list(range(n))
    assert jd_col.tolist() == [-1] * 5 and jd_val.tolist() == [7.0] * 5
