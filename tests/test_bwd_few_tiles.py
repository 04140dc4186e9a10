"""GPU parity of the backward on both sides of the rules that pick its dK/dV and dQ kernels by the
number of tiles: few tiles (32 keys or queries per workgroup, dealt out to its waves) and many (128 per
workgroup).  Bound and oracle as in test_bwd_parity."""
import pytest

from test_bwd_parity import check_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La", [(1, 1, 1, 1, 64, 2, 3), (1, 2, 1, 31, 128, 5, None), (2, 2, 2, 32, 64, 6, None),
                                              (1, 4, 1, 33, 128, 3, 4), (1, 6, 2, 127, 64, 0, None), (1, 3, 3, 129, 128, 11, 12),
                                              (1, 10, 2, 161, 64, 4, None), (1, 9, 1, 97, 128, 2, None)])
def test_bwd_few_tiles(B, Hq, Hk, T, d, L, La, causal):
    check_full(B, Hq, T, d, L, 1300 + T + L, causal=causal, depth_alloc=La, Hk=Hk)


@pytest.mark.parametrize("B,Hq,Hk,T,d,L,La,causal", [(89, 8, 8, 130, 64, 5, 6, True), (89, 16, 8, 131, 64, 3, None, True),
                                                     (45, 32, 8, 190, 64, 2, 3, True), (24, 16, 8, 257, 128, 6, None, False),
                                                     (24, 64, 16, 65, 128, 1, 2, True), (24, 40, 8, 130, 64, 2, None, False)])
def test_bwd_many_tiles_of_short_sequences(B, Hq, Hk, T, d, L, La, causal):
    """Enough (batch, head) pairs for the kernels of 128 keys / queries per workgroup."""
    check_full(B, Hq, T, d, L, 1400 + T + L, causal=causal, depth_alloc=La, Hk=Hk)
