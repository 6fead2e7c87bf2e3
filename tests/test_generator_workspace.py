"""The generator backward's scratch: r_in, h and dpre of every token and one partial of all weight gradients per 256 tokens,
each part rounded up to 256 bytes.  A caller may have sized its buffer by that, so it must not grow."""
import pytest

from paper_2603_06738_amd import binding as rb


@pytest.mark.parametrize("M,heads,r,L,d_h", [(1, 1, 1, 0, 1), (16, 6, 18, 10, 32), (17, 2, 5, 3, 33), (48, 3, 16, 10, 32),
                                             (96, 6, 34, 10, 32), (256, 64, 64, 16, 64)])
def test_scratch_does_not_grow(M, heads, r, L, d_h):
    N, n_in, up = M * M, 2 + 4 * L, lambda x: (x + 255) // 256 * 256
    elems = 2 * heads * d_h * r + n_in * d_h + d_h
    most = up(N * n_in * 4) + 2 * up(N * d_h * 4) + up((N + 255) // 256 * elems * 4)
    assert 0 < rb.rib_features_bwd_workspace_bytes(rb.make_gen_params(M, heads, r, L, d_h)) <= most
