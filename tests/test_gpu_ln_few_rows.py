"""GPU parity of LayerNorm at the row counts where its kernels change: narrow rows from 1536 on take a wavefront each, wide rows up
to two per compute unit (512 here; of float rows of more than 8192 one, 256) take 512 threads with every load ahead of the sums.  Checks and bounds of the narrow rows."""
import pytest

import test_gpu_ln_narrow as narrow

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,H", [(1535, 512), (1536, 512), (1537, 1024), (1536, 1032), (2051, 8), (1, 4104), (512, 4104), (513, 4104), (511, 8200), (256, 8200), (257, 8200),
                                 (5, 16384), (130, 12296)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_few_rows(dtype, M, H):
    narrow.test_narrow_rows(dtype, M, H)
