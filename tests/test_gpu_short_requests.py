"""GPU parity of batches of short requests, at the sizes where the sharing rule
changes how it counts them: around the limit below which a request counts for
more than its bytes, with empty ones, and with one long request among many
short ones; in the kernel's arguments (up to 256 requests), in pinned memory,
and over a scanned table.  Whole pool and all counters against the oracle, for
submissions and plan replays."""
import pytest

from tests.test_gpu_stream import gpu, test_batch_sizes as _batch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 64, 65, 256, 257, 1024, 4096, 4097, 9000])
@pytest.mark.parametrize("sizes", [[1], [1023, 1024, 1025, 0], [8] * 127 + [300_001]])
def test_short_requests(gpu, n, sizes):  # noqa: F811
    _batch(gpu, n, sizes)
