"""elora_batched_lora_linear_noalloc over changes of d_out: the one array serves each call's mailboxes in their idle state,
whatever calls of other kernels and other d_out have written into it before.  Calls of 65 to 256 rows on a large W may run
as launches of the decode kernel here and as one product with a workspace (the array does not always hold the sums of the
latter), so those are compared with the oracle alone."""
import numpy as np
import pytest
import torch

from gpu_harness import DeviceCase, assert_close, y_to_f64
from paper_2507_01438_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_alternating_d_out_after_calls_that_fill_the_array():
    from paper_2507_01438_amd import binding as B
    # (T, K, N, the workspace call runs the same kernels)
    shapes = [(64, 2048, 1040, True), (700, 2048, 2048, True), (40, 1024, 272, True), (150, 2048, 2064, False), (33, 4096, 4096, True), (9, 100, 30, True),
              (90, 1088, 264, True), (256, 4096, 1040, False)]
    cases = [DeviceCase(w, w.projections[0]) for w in (I.small_workload(970 + i, I.BF16, K, N, T, 5, (8, 16, 32, 64), no_adapter_rows=(1,)) for i, (T, K, N, _) in enumerate(shapes))]
    want = [c.run() for c in cases]
    order = list(range(len(cases))) * 2 + [1, 0, 1, 4, 1, 2, 3, 0, 7, 5, 4, 4, 3, 3]
    for i in order:
        c = cases[i]
        c.y.fill_(7)
        d = c.desc()
        d.workspace, d.workspace_bytes = None, 0
        B.elora_batched_lora_linear_noalloc(d)
        torch.cuda.synchronize()
        y = y_to_f64(c.y[: c.w.T], I.BF16)
        if shapes[i][3]:
            np.testing.assert_array_equal(y, want[i], err_msg=str(shapes[i]))
        else:
            assert_close(y, c.reference(), c.base_reference(), str(shapes[i]))
    for c in cases:
        assert c.pool.poll_error() == (0, -1)
        c.close()
