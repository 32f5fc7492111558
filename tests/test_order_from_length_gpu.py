"""The order by length starts at caches of 512 keys, and at 40 keys a sequence in
large batches: prefill batches on both sides of that equal, bit for bit, each
sequence's own call."""
import pytest

from test_order_by_length_gpu import test_prefill_sequences_equal_their_own_calls as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [(2, 64, 16, 300, 511, 64, True, "bf16"), (2, 64, 16, 300, 512, 64, True, "bf16"),
                                  (7, 64, 8, 200, 733, 128, True, "bf16"), (64, 4, 2, 300, 1279, 64, True, "bf16"),
                                  (64, 4, 2, 300, 1280, 64, True, "bf16"), (64, 4, 2, 300, 2559, 64, True, "bf16"),
                                  (64, 4, 2, 300, 2560, 64, True, "bf16"), (16, 16, 16, 33, 639, 64, True, "f16"),
                                  (16, 16, 16, 33, 640, 128, True, "f16"), (9, 32, 8, 150, 600, 128, False, "f16"),
                                  (65, 4, 2, 300, 1310, 64, True, "f16"), (40, 16, 16, 33, 800, 128, True, "f16")],
                         ids=lambda c: "x".join(map(str, c)))
def test_both_sides(case):
    check(case)
