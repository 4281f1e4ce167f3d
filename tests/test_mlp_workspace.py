"""The trainer's workspace holds what training works on (weights, gradient and
two moments of 5,313 floats, the block sums of the gradient, at most 256 of
5,314 floats, mean and std, two losses), whatever the batch: no row's
activations are stored."""
from paper_2608_22269_amd import _lib as L


def test_workspace_does_not_grow_with_the_batch():
    lib = L.lib()
    most = 4 * (4 * 5313 + 256 * 5314 + 2 * 16 + 2) + 16 * 256  # each array at a multiple of 256 bytes
    sizes = [lib.sph_mlp_workspace_bytes(b) for b in (1, 8, 9, 1000, 2048, 2049, 4096, 1 << 20, 1 << 24)]
    assert all(0 < s <= most for s in sizes), sizes
    assert sizes == sorted(sizes) and sizes[4] == sizes[-1]
    assert lib.sph_mlp_workspace_bytes((1 << 24) + 1) == 0 and lib.sph_mlp_workspace_bytes(0) == 0
