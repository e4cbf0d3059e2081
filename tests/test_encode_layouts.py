"""The lane layout that the encoder takes for a call (nothing runs): few tokens of many sequences stay with the layout of small
calls, as their number fills neither the waves nor the workgroups of the sixteen-channel layout; long prompts take that one."""
import os

import pytest

from paper_2505_18231_amd import api
from tests import helpers

FORMATS = [(4, False, False, 16, 0), (4, False, True, 16, 0), (4, False, False, 4, 0), (4, False, False, 16, 64), (8, False, False, 16, 0),
           (8, True, False, 16, 0), (8, False, True, 16, 0), (8, True, True, 4, 64)]  # sub_dim, sign, rope, side_bits, group


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(api.LIB_PATH):
        from paper_2505_18231_amd.build import build_library
        build_library(verbose=False)


def _layout(fmt, batch, kv_heads, max_new):
    sub, sign, rope, side_bits, group = fmt
    shape = api.make_shape(sub, kv_heads, kv_heads, 1 << 17, group, 0, sign_format=sign, side_bits=side_bits)
    shape.rope_table = 4096 if rope else None  # (looked at as a flag)
    return helpers.encode_layout(api, shape, batch, max_new)


@pytest.mark.parametrize("fmt", FORMATS)
def test_few_tokens_of_many_sequences_keep_the_layout_of_small_calls(fmt):
    sub = fmt[0]
    for batch in (1, 48, 64, 75, 128, 192, 384, 512, 768, 1000, 4096, 60000):
        for kv_heads in (1, 8, 32):
            for max_new in (1, 2):
                assert _layout(fmt, batch, kv_heads, max_new) == sub, (batch, kv_heads, max_new)
            for max_new in range(3, 17 if sub == 8 else 9):
                assert _layout(fmt, batch, kv_heads, max_new) != 16, (batch, kv_heads, max_new)


@pytest.mark.parametrize("fmt", FORMATS)
def test_long_prompts_take_sixteen_channels_and_short_ones_the_shortest_chain(fmt):
    for batch, kv_heads, max_new in ((8, 8, 8192), (1, 8, 131072), (4, 8, 4096), (32, 32, 1024), (64, 8, 64)):
        assert _layout(fmt, batch, kv_heads, max_new) == 16, (batch, kv_heads, max_new)
    for batch, kv_heads, max_new in ((1, 1, 1), (1, 8, 64), (4, 8, 64), (1, 8, 256), (256, 1, 8)):
        assert _layout(fmt, batch, kv_heads, max_new) == fmt[0], (batch, kv_heads, max_new)


def test_eight_channels_lie_between_them():
    for batch, kv_heads, max_new in ((9, 8, 64), (16, 8, 32), (65, 8, 9), (1, 8, 500)):
        assert _layout(FORMATS[0], batch, kv_heads, max_new) == 8, (batch, kv_heads, max_new)
    for fmt in FORMATS[2:]:  # (an instance of the plain 4-dim formats)
        for batch in range(1, 200):
            assert _layout(fmt, batch, 8, 64) in (fmt[0], 16)


def _form(fmt, batch, kv_heads, max_new):
    sub, sign, rope, side_bits, group = fmt
    shape = api.make_shape(sub, kv_heads, kv_heads, 1 << 17, group, 0, sign_format=sign, side_bits=side_bits)
    shape.rope_table = 4096 if rope else None
    return helpers.encode_launch_form(api, shape, batch, max_new)


@pytest.mark.parametrize("fmt", FORMATS)
def test_ragged_batches_take_three_workgroups_to_a_unit_only_where_they_are_many(fmt):
    """A batch's places need not hold tokens: with few of them, three workgroups with tokens would share one compute unit while others
    have none.  One sequence fills its places: there the rounds of the chip decide."""
    for batch, kv_heads, max_new in ((16, 1, 1088), (8, 4, 640), (8, 4, 1664), (31, 1, 1056), (2, 8, 4032)):
        layout, tokens, units = _form(fmt, batch, kv_heads, max_new)
        assert 512 < 2 * kv_heads * batch * -(-max_new // tokens) < 2048
        assert layout == 16 and units == 2, (batch, kv_heads, max_new, layout, units)
    for batch, kv_heads, max_new in ((2, 8, 4096), (16, 2, 2048), (32, 1, 2048), (8, 8, 8192)):
        layout, tokens, units = _form(fmt, batch, kv_heads, max_new)
        assert layout == 16 and units == 3, (batch, kv_heads, max_new, layout, units)
    for places, want in ((512, 2), (513, 3), (768, 3), (769, 2), (1024, 2), (1025, 3), (4000, 3)):
        # (one kv head: an even number of places, in 64-token workgroups below half a million token places)
        max_new = 64 * ((places + 1) // 2 if want == 3 or places > 768 else places // 2)
        layout, tokens, units = _form(fmt, 1, 1, max_new)
        assert (layout, tokens, units) == (16, 64, want), (places, layout, tokens, units)
