"""Scratch of calls without a workspace: which of them share a block (host logic, no GPU)."""
import threading

import torch

from paper_2506_11449_amd.binding import DefaultBlocks

new = lambda n: torch.empty(n, dtype=torch.uint8)


def test_a_block_for_each_stream_grown_on_demand():
    blocks = DefaultBlocks()
    a, b = blocks.get(("dev", 1), 100, new), blocks.get(("dev", 2), 100, new)
    assert a.data_ptr() != b.data_ptr()
    assert blocks.get(("dev", 1), 60, new) is a
    larger = blocks.get(("dev", 1), 101, new)
    assert larger.numel() == 101 and blocks.get(("dev", 1), 100, new) is larger and blocks.get(("dev", 2), 100, new) is b


def test_a_block_for_each_thread():
    blocks, seen = DefaultBlocks(), []
    mine = blocks.get("stream", 100, new)
    worker = threading.Thread(target=lambda: seen.append(blocks.get("stream", 100, new)))
    worker.start()
    worker.join()
    assert seen[0].data_ptr() != mine.data_ptr() and blocks.get("stream", 100, new) is mine


def test_the_oldest_blocks_are_given_up():
    blocks = DefaultBlocks()
    for i in range(3 * DefaultBlocks.MOST):
        blocks.get(i, 10, new)
        assert len(blocks.blocks) <= DefaultBlocks.MOST
    assert set(blocks.blocks) == set(range(2 * DefaultBlocks.MOST, 3 * DefaultBlocks.MOST))
