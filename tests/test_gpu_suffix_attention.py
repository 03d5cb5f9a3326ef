"""The action expert's attention kernel (16 query rows per block) at the edges of what it takes: prefixes shorter than a
16-key tile, ending inside one, exactly full shares, and every way of sharing out the values."""
import pytest

from tests import test_gpu_attention as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,chunks_per_share", [(1, 0), (15, 0), (17, 0), (225, 0), (256, 0), (257, 8), (512, 8), (300, 3), (1024, 8)])
@pytest.mark.parametrize("v_split", [1, 2, 4, 8])
def test_prefix_lengths_and_value_splits(P, chunks_per_share, v_split):
    base.test_expert_attention_block_mask_and_key_shares(P, chunks_per_share, v_split)


# a ninth and a tenth chunk, each with its first 16-key tile only, ending inside a tile, and full; the last share with fewer
@pytest.mark.parametrize("P,chunks_per_share", [(257, 0), (271, 0), (288, 0), (290, 0), (305, 0), (320, 0), (530, 9), (561, 9), (625, 10), (816, 9)])
@pytest.mark.parametrize("v_split", [1, 2, 8])
def test_shares_of_nine_and_ten_chunks(P, chunks_per_share, v_split):
    base.test_expert_attention_block_mask_and_key_shares(P, chunks_per_share, v_split)


# the prefix's own attention, any number of query rows over up to ten chunks, and one row more than this kernel takes
@pytest.mark.parametrize("P", [1, 17, 31, 33, 255, 257, 273, 288, 320, 321])
def test_prefix_of_up_to_ten_chunks(P):
    base.test_prefix_attention_shared_head(P)
