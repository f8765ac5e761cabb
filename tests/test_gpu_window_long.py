"""Windows whose ring of messages would not fit the LDS, but whose two sums per
variable do: messages in registers, bit for bit as the launch-per-phase form."""
import pytest

import test_gpu_window

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,positions,W,K,gamma,terminate", [(512, 20, 8, 2, 2, True), (512, 14, 12, 2, 3, False),
                                                             (320, 22, 18, 2, 2, True), (100, 40, 36, 2, 2, True)])
def test_long_windows(p, positions, W, K, gamma, terminate):
    test_gpu_window.test_register_and_launch_paths_agree_bit_for_bit(p, positions, W, K, gamma, terminate)


@pytest.mark.parametrize("p,positions,W,K,gamma,terminate", [(513, 9, 6, 2, 3, True), (600, 8, 3, 3, 300, False),
                                                             (700, 7, 5, 2, 2, True), (900, 9, 4, 2, 3, True),
                                                             (1023, 9, 6, 2, 2, False)])
def test_long_circulants(p, positions, W, K, gamma, terminate):
    test_gpu_window.test_register_and_launch_paths_agree_bit_for_bit(p, positions, W, K, gamma, terminate)
