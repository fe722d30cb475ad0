"""Filter and bias gradients of layers that read the caller's input directly, are narrower than a matrix-core block, or have a
bias: every such gradient against the oracle (sizes large enough for the matrix-core kernels, see wgrad_wide_enough)."""
import pytest

from ftp_synth.configs import Config, conv, pool
from tests import parity as P

pytestmark = pytest.mark.gpu

_NETS = {
    "pooled": ((conv(32, 64), pool(64)), 48, 64),
    "plain": ((conv(40, 48), conv(48, 24)), 30, 46),
    "narrow": ((conv(16, 24), conv(24, 12), conv(12, 8)), 66, 70),
    # odd strides between channels and between images: rows of 16-bit maps that start between dwords
    "oddchannels": ((conv(3, 9), conv(9, 16)), 33, 45),
    "oddpool": ((conv(3, 8), conv(8, 9), pool(9)), 66, 70),
    "oddcaller": ((conv(72, 16, 1), conv(16, 32)), 31, 31),
    "oddwidth": ((conv(16, 40), conv(40, 32)), 33, 45),
    "other": ((conv(24, 20, 5), conv(20, 12, 1), conv(12, 16, 3, stride=2)), 62, 58),
}


@pytest.mark.parametrize("net", sorted(_NETS))
@pytest.mark.parametrize("dtype,bias", [("bf16", False), ("f32", False), ("f32", True), ("bf16", True)])
@pytest.mark.parametrize("grid", [(1, 1), (2, 3)])
def test_gradients(oracle, net, dtype, bias, grid):
    layers, h, w = _NETS[net]
    P.check_case(oracle, Config("routes_" + net, 3, layers[0].cin, h, w, layers, grid, (len(layers),), dtype), has_bias=bias)
