"""What bench.py divides by a launch's time: logits rows that are computed and read, not rows of codes."""
import numpy as np

import bench


def test_rows_of_a_decode_with_and_without_sharing():
    # 2 prompts x 3 codes, 4 steps, EOS = 1: two rows end after their second token
    tokens = np.array([[[5, 5, 7, 7], [5, 1, 1, 1], [6, 6, 7, 9]],
                       [[5, 8, 8, 8], [9, 1, 1, 1], [6, 6, 8, 9]]])
    own = bench.step_counts(tokens, 1, 2, False)
    assert own == {"active": (6 + 6 + 4 + 4) / 4, "computed": (2 + 6 + 6 + 6) / 4, "fetched": (2 + 6 + 4 + 4) / 4}
    # tokens conditioned on: {5, 6, 9}, {5, 1, 6, 8}, {7, 1, 8}; by rows still running the last two lose EOS
    shared = bench.step_counts(tokens, 1, 2, True)
    kept = bench.step_counts(tokens, 1, 2, False, True)
    assert kept == {"active": 5.0, "computed": (2 + 3 + 3 + 0) / 4, "fetched": (2 + 3 + 3 + 2) / 4}
    assert shared == {"active": 5.0, "computed": (2 + 3 + 4 + 3) / 4, "fetched": (2 + 3 + 3 + 2) / 4}


def test_rows_are_kept_where_most_come_again():
    def kept(V, d, R, T, by_sums=True):
        return bench.rows_kept(V, d, R, 1, T, "bf16", V * 2, by_sums)
    assert kept(32128, 512, 65536, 16) and kept(32128, 512, 8192, 4) and kept(8000, 512, 4096, 4) and kept(2000, 128, 2048, 64)
    assert not kept(32128, 512, 1024, 64) and not kept(8000, 512, 2048, 16) and not kept(2000, 128, 1024, 64)
    # a vocabulary of more than four times the rows: over three or four steps
    assert kept(32128, 512, 8000, 4) and not kept(32128, 512, 8000, 5) and kept(32128, 512, 8192, 5)
    assert not kept(5001, 512, 2048, 16, False) and kept(5001, 512, 2048, 64, False)


def test_sharing_pays_for_wide_lattices_only():
    def shared(V, d, R, T=16, wdt="bf16"):
        return bench.rows_shared(V, d, R, T, wdt, 256)
    assert shared(32128, 512, 65536) and shared(32128, 512, 6700) and shared(4096, 512, 12288)
    assert not shared(32128, 512, 1024) and not shared(32128, 512, 65536, T=1) and not shared(32128, 512, 65536, wdt="f32")
    # the rows in use leave workers of the product without a row tile
    assert not shared(32128, 512, 8192) and not shared(32128, 1024, 6144)


def test_rows_of_an_encode():
    # conditioned on: the prompts 3, 4, then 5 and 6 (rows that have not ended), 7 once
    seqs = np.array([[5, 7, 9], [1, 8, 8], [6, 1, 8], [5, 7, 1]])
    assert bench.conditioned_tokens(seqs, np.array([3, 4]), 1) == 5
    assert bench.conditioned_tokens(seqs, np.array([3, 4]), -1) == 7
