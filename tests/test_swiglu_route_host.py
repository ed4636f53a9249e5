"""How the two SwiGLU projections are launched alone on the GPU: in which tile together, or apart."""
import pytest

import paper_2510_27257_amd as stp


# tokens, hidden, ffn: narrow tiles where few tokens leave the wide ones half empty; apart where a tile of both is too slow for the rounds
# it fills; the shards of the workloads together; outputs of the contraction-splitting kernel apart
@pytest.mark.parametrize("T,h,f,tile", [(136, 5120, 14336, (128, 256)), (136, 7168, 14336, (128, 256)), (136, 520, 14336, (128, 256)),
                                        (520, 4096, 14336, None), (1032, 5120, 8192, None), (1544, 7168, 5120, (192, 256)),
                                        (4096, 7168, 5120, (256, 256)), (4096, 5120, 3456, (256, 256)), (3072, 5120, 1728, (192, 256)),
                                        (264, 512, 1024, None)])
def test_route(T, h, f, tile):
    got = stp.lib().stp_swiglu_pair_tile(T, f, h)
    assert (got >> 16, got & 0xffff) == (tile or (0, 0))
