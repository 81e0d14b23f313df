"""The drafter layer around the token counts where its launches change: K, V
and q in one launch up to 16 tokens, W_o and W_down with their residual in one
kernel up to 11 tokens on layers of at least 256 feature blocks (4096).
Against the fp64 oracle, with the bf16 bar of the other drafter tests."""
import pytest

from test_gpu_drafter import test_forward_matches_oracle as check_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 2, 11, 12, 16, 17])
@pytest.mark.parametrize("hidden,nqh,nkvh,hd,inter,pos", [
    (4096, 2, 1, 128, 96, 40),           # exactly 256 feature blocks, short inputs
    (4128, 5, 5, 64, 352, 0),            # more, none a power of two
    (4064, 4, 2, 64, 128, 9),            # 254 blocks: the slices
])
def test_forward_rows(hidden, nqh, nkvh, hd, inter, pos, M):
    check_forward(hidden, nqh, nkvh, hd, inter, pos, M)
