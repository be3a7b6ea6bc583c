"""Chunk lengths of the attention backward pass, seen in the workspace it asks for.  No GPU needed (the rule then counts on 256 compute units,
an MI355X's)."""
import pytest

from paper_2411_15871_amd import dhelix as dh


# dQ in whole rows, whose longest blocks end by themselves and faster, is the shorter launch here (16:2 heads x 5000 tokens: 102 us, in chunks of 68 tiles
# 120): the workspace holds the row statistics and the partial dK, dV of key blocks cut into chunks of dkv_tiles, and no partial dQ.
@pytest.mark.parametrize("batch,seq,nq,nkv,dkv_tiles", [(1, 5000, 16, 2, 52), (3, 2727, 8, 2, 24), (1, 7000, 32, 4, 202)])
def test_whole_rows_have_no_dq_partials(batch, seq, nq, nkv, dkv_tiles):
    d, stats = 64, -(-nq * batch * seq * 4 // 256) * 256
    tiles = [nq // nkv * ((seq - i + 63) // 64) for i in range(0, seq, 128)]  # of a key block: its group's heads, one after the other
    partials = batch * nkv * sum(-(-t // dkv_tiles) for t in tiles) * 128 * 2 * d * 4
    assert dh.dh_attn_bwd_workspace_bytes(dh.DH_BF16, batch, seq, nq, nkv, d) == stats + partials


# Over more than 1024 key blocks no block is cut, however many tiles its head group has (more than 2^20 here): were a length left that such blocks exceed, the
# launch would count their chunks, and the kernel, which takes every unit for a whole block, would walk blocks behind the last one.
@pytest.mark.parametrize("seq,nq,d", [(1100000, 64, 64), (1100000, 64, 128), (4300000, 16, 64)])
def test_blocks_of_very_long_head_groups_stay_whole(seq, nq, d):
    stats = -(-nq * seq * 4 // 256) * 256
    assert nq * (-(-seq // 64)) > 1 << 20
    assert dh.dh_attn_bwd_workspace_bytes(dh.DH_BF16, 1, seq, nq, 1, d) == stats


# Behind a key buffer a query block's row has many times the tiles of a key block's columns.  Equal heads are cut alike, by the longer of the two: the workspace holds
# partial dQ of at least eight chunks a row (176 us with whole rows of 125 tiles, 36 in chunks of 14) and, the columns being shorter than a chunk, no partial dK, dV.
@pytest.mark.parametrize("batch,seq,q_off,heads,d", [(1, 189, 7808, 4, 128), (1, 141, 6912, 1, 128), (1, 238, 6016, 1, 64), (4, 187, 2048, 1, 128)])
def test_rows_behind_a_key_buffer_are_cut(batch, seq, q_off, heads, d):
    stats, blocks = -(-heads * batch * seq * 4 // 256) * 256, (q_off + seq + 127) // 128 - q_off // 128
    partial = dh.dh_attn_ctx_bwd_workspace_bytes(dh.DH_BF16, batch, seq, q_off, heads, heads, d) - stats
    units, rest = divmod(partial, batch * heads * 128 * d * 4)
    assert rest == 0 and units >= 8 * blocks, (units, blocks)
    chunk = next(c for c in range(2, 1 << 20, 2) if sum(-(-((min((i + 1) * 128, q_off + seq) + 63) // 64) // c) for i in range(q_off // 128, q_off // 128 + blocks)) <= units)
    assert chunk >= (seq + 63) // 64  # the longest column


# The key blocks of a few short sequences are fewer than the compute units, and each walks its whole head group: cut into chunks of two tiles (4:2 heads x 224 tokens
# 32.6 -> 26 us, a block per query head 29).
@pytest.mark.parametrize("batch,seq,nq,nkv,d", [(1, 224, 4, 2, 128), (1, 233, 16, 8, 128), (1, 145, 32, 8, 64), (2, 386, 8, 4, 64)])
def test_short_head_groups_are_cut(batch, seq, nq, nkv, d):
    stats = -(-nq * batch * seq * 4 // 256) * 256
    units = sum(-(-(nq // nkv * ((seq - i + 63) // 64)) // 2) for i in range(0, seq, 128))
    assert dh.dh_attn_bwd_workspace_bytes(dh.DH_BF16, batch, seq, nq, nkv, d) == stats + batch * nkv * units * 128 * 2 * d * 4


# Equal heads of 64: enough whole rows and columns to fill the units twice are faster than shorter ones with partial results (8 heads x 2 x 1660 tokens 45 us, cut into
# 14 tiles 50).
@pytest.mark.parametrize("batch,seq,heads", [(2, 1660, 8), (2, 1400, 8), (2, 2048, 8)])
def test_equal_narrow_heads_that_fill_the_chip_stay_whole(batch, seq, heads):
    assert dh.dh_attn_bwd_workspace_bytes(dh.DH_BF16, batch, seq, heads, heads, 64) == -(-heads * batch * seq * 4 // 256) * 256
