"""How far the host loop of a solve runs ahead of its status reads (hmc_test_chunks, simulated records):
no chunk is issued past the end of a solve whose records told how much was left, whether the host had
waited before or not."""
import itertools

import pytest

from paper_2204_14241_amd import hmc

NEEDS = [1, 7, 31, 32, 33, 60, 64, 65, 90, 100, 129, 500, 2344]


@pytest.mark.parametrize("free_len", [False, True])
@pytest.mark.parametrize("chunk", [32, 50, 96])
def test_no_chunk_past_a_known_end(chunk, free_len):
    for need, last in itertools.product(NEEDS, [0] + NEEDS):
        issued, idle, waits = hmc.test_chunks(need, 0, last, chunk, free_len)
        # one chunk past the end only where the first chunk ends the solve and no estimate said so
        assert idle == (1 if need <= chunk and (last == 0 or last > chunk) else 0), (need, last)
        least = (need + chunk - 1) // chunk
        assert issued - idle == least if not free_len else least <= issued - idle <= least + 1, (need, last)
        assert waits <= 2


@pytest.mark.parametrize("free_len", [False, True])
@pytest.mark.parametrize("bias", [-40, -3, 3, 40])
def test_wrong_estimates(bias, free_len):
    for need, last in itertools.product(NEEDS, [0] + NEEDS):
        issued, idle, waits = hmc.test_chunks(need, bias, last, 50, free_len)
        assert idle <= 1


@pytest.mark.parametrize("k0", [2, 4])
def test_after_a_step_graph(k0):
    # the graph's chunks were read: what follows is sized by those records
    for more in (1, 20, 31, 50, 51, 99, 100, 260):
        issued, idle, waits = hmc.test_chunks(50 * k0 + more, 0, 77, 50, False, k0)
        assert (issued, idle) == ((more + 49) // 50, 0)
