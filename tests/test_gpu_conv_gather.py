"""The 3 x 3 convolutions gathered tap by tap inside the product (channel counts
that are multiples of 64: no im2col matrix), forward and input gradient, through a
ResNet step against the oracle (run_parity's bounds): maps of 1 x 1 up to 18 x 18
pixels, odd and even (padding on every side, a tile's rows in several images),
strides 1 and 2, a last row tile that ends inside a tile, and pixel counts that
are no multiple of 8."""

import pytest

from tests.test_gpu_resnet import run_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("img,batch,blocks", [(32, 3, (2, 1, 1, 2)), (72, 5, (2, 2, 1, 1)), (56, 7, (1, 2, 2, 1))])
def test_gathered_convolutions(img, batch, blocks):
    run_parity(dict(arch="resnet", n_layers=sum(blocks), res_blocks=blocks, res_width=64, vocab=30, img_size=img,
                    channels=3, batch=batch, lr=1e-4), steps=1)
