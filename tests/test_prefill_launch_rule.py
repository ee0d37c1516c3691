"""The prefill launch rule, on the host (no GPU): which of its launch shapes a
call takes.

  * The launch-shape tests on the GPU take every shape at every k.
  * Calls that an earlier rule slowed down (it took a shape whose workgroups a
    CU holds one at a time for one that shares it, and had none for a single
    group over many tokens) take a shape that is fast for them.
  * The longest prompts have a shape whose grid they fit.
"""
import ctypes as C

import pytest

import paper_2509_18172_amd as sb
from test_gpu_prefill import SHAPE_CASES

LIB = C.CDLL(sb.library_path())
# Indices of the rule's table: the 16-row kernel's shapes (8 wavefronts, 16
# wavefronts, 32-token tiles), then by (column tiles, token tiles, row groups).
SHORT, SHORT_16_WAVES, SHORT_32_TOKENS = 0, 1, 2
SHAPES = [(1, 1, 1), (1, 2, 1), (1, 2, 2), (1, 2, 4), (1, 4, 2), (1, 4, 4), (1, 4, 8), (1, 1, 8), (2, 4, 8)]


def shape(O, I, k, T):
    return LIB.sbvr_test_prefill_shape(O, I, k, T)


def index(*s):
    return 3 + SHAPES.index(s)


@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_shape_cases_take_every_shape(k):
    n = LIB.sbvr_test_prefill_shapes()
    assert n == 3 + len(SHAPES)
    assert {shape(O, I, k, T) for O, I, T in SHAPE_CASES} == set(range(n))
    # the 16-wavefront shape with all sixteen at work: a full token tile, a
    # partial one, and tiles with a remainder
    full = [T for O, I, T in SHAPE_CASES if I // 128 >= 16 and shape(O, I, k, T) == SHORT_16_WAVES]
    assert any(T % 16 == 0 for T in full) and any(T < 16 for T in full) and any(T > 16 and T % 16 for T in full)


# Times on MI355X of the calls a rule that ignored the rounds sent to the 32-token
# tiles of the 16-row kernel, whose workgroups a CU holds one at a time: 16.2, 9.7
# and 10.3 us; the best shapes take 8.5, 7.4 and 6.7.
@pytest.mark.parametrize("O,I,k,T", [(18332, 896, 2, 23), (12011, 1024, 2, 26), (10710, 896, 1, 25)])
def test_rounds_count(O, I, k, T):
    assert shape(O, I, k, T) != SHORT_32_TOKENS


# 6.6, 5.8 and 5.4 us with several K-slices or 128-token tiles, 4.1, 3.9 and 3.7
# with a single K-slice and 32 tokens.
@pytest.mark.parametrize("O,T", [(6599, 265), (14088, 107), (8344, 91)])
def test_single_groups_over_many_tokens(O, T):
    assert shape(O, 128, 1, T) == index(1, 1, 8)


def test_longest_prompts_have_a_shape():
    """2^22 tokens, the most sbvr_gemm_prefill takes: a grid's second dimension
    holds their tiles in every shape that is taken."""
    tokens = [16, 16, 32] + [32 * tt for _, tt, _ in SHAPES]
    for O, I in ((1, 128), (16, 4096), (511, 4194176)):
        for T in (1, 1 << 20, (1 << 22) - 1, 1 << 22):
            s = shape(O, I, 4, T)
            assert 0 <= s < len(tokens) and -(-T // tokens[s]) <= 65535
