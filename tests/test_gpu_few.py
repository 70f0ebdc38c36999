"""Tiles of a few elements off the vector grid, which an all-kinds launch
copies one element per lane: biases of 63 to 65 elements per shard (the most a
wavefront takes, and one more), strided boxes of a few columns, and boxes whose
padding is all but one of eight elements; every byte against the oracle, with
and without direct Refer."""
import pytest

from paper_2607_04749_amd.workloads import GPT, ModelShape, Parallel as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ffn", [2, 18, 126, 128, 130])
@pytest.mark.parametrize("src,dst", [(P(1, 1), P(2, 1)), (P(2, 1), P(1, 2))])
@pytest.mark.parametrize("direct_refer", [False, True])
def test_boxes_of_a_few_elements(ffn, src, dst, direct_refer):
    from gpu_util import full_compare
    model = ModelShape(GPT, 2, 6, 2, 2, ffn, 10, 3, 1)
    print("[gpu] few elements: ffn", ffn, src, "->", dst, "refer", direct_refer, flush=True)
    full_compare(model, src, dst, 0xF0 + ffn, direct_refer=direct_refer)
