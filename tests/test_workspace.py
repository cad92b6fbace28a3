"""Scratch of the sequence model's training steps in fp32: copies of the weights for split products are kept only by batches whose
products gain from them.  Everything else grows linearly with the batch."""
import pytest


@pytest.fixture
def bls():
    import paper_2508_08540_amd as bls
    return bls


def _jump(bls, batch, *model):
    """Bytes by which the scratch of `batch` sequences exceeds what the two smaller batches let expect."""
    m = bls.Model.transformer(*model)
    w = [m.workspace_bytes(batch - i, True) for i in range(3)]
    return (w[0] - w[1]) - (w[1] - w[2])


@pytest.mark.parametrize("vocab,D,H,F", [(1000, 64, 2, 256), (1000, 128, 4, 512), (1000, 256, 8, 1024)])
def test_narrow_encoders_of_512_tokens_keep_no_copies(bls, vocab, D, H, F):
    weights = 2 * (4 * D * D + 2 * D * F) + vocab * D
    assert abs(_jump(bls, 4, vocab, 128, D, H, F, 2)) < 6 * weights   # one copy in three bf16


@pytest.mark.parametrize("vocab,D,H,F,batch", [(32000, 64, 2, 256, 4), (1000, 256, 8, 1024, 17), (1000, 512, 8, 2048, 5)])
def test_larger_products_keep_two_copies(bls, vocab, D, H, F, batch):
    weights = 2 * (4 * D * D + 2 * D * F) + vocab * D
    sizes = [bls.Model.transformer(vocab, 128, D, H, F, 2).workspace_bytes(b, True) for b in (2, 3, batch)]
    assert sizes[2] - sizes[1] - (batch - 3) * (sizes[1] - sizes[0]) > 12 * weights


def test_no_copy_of_the_vocabulary_projection_that_no_product_reads(bls):
    """Rows of 32 001 logits do not start on 16 bytes, so the input gradient of the projection keeps the fp32 instruction."""
    layers = 2 * (4 * 512 * 512 + 2 * 512 * 2048)
    extra = {}
    for vocab in (32000, 32001):
        extra[vocab] = _jump(bls, 4, vocab, 128, 512, 8, 2048, 2)
    assert extra[32000] >= 12 * (layers + 32000 * 512)
    assert extra[32000] - extra[32001] >= 5 * 32000 * 512
