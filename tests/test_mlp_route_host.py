"""Which networks take the block kernel shows in the workspace they ask for: one gradient
buffer a layer there, two in all layer by layer."""
import pytest

from paper_1305_1183_amd import kf


def floats(d, h, L, n):
    m = kf.kf_mlp_create(d, h, L)
    b = kf.kf_mlp_workspace_bytes(m, n)
    kf.kf_mlp_destroy(m)
    return b // 4


@pytest.mark.parametrize("d,h,L,n,block", [(32, 128, 3, 256, True), (32, 128, 4, 1, True), (480, 96, 8, 16, True),
                                           (480, 480, 16, 16, False), (32, 200, 4, 16, False), (33, 300, 4, 64, False),
                                           (8, 129, 5, 4095, False), (8, 129, 5, 4096, True), (480, 480, 8, 32768, True),
                                           (481, 64, 4, 32768, False)])
def test_few_samples_of_a_wide_network_go_layer_by_layer(d, h, L, n, block):
    assert floats(d, h, L, n) == (2 * L if block else L + 2) * n * h + 2 * n + 64
