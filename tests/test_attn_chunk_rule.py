"""Chunk lengths of the attention backward pass, seen in the workspace it asks for.  No GPU needed (the rule then counts on 256 compute units,
an MI355X's)."""
import pytest

from paper_2411_15871_amd import dhelix as dh


# dQ in whole rows, whose longest blocks end by themselves and faster, is the shorter launch here (16:2 heads x 5000 tokens: 102 us, in chunks of 68 tiles
# 120): the workspace holds the row statistics and the partial dK, dV of key blocks cut into chunks of dkv_tiles, and no partial dQ.
@pytest.mark.parametrize("batch,seq,nq,nkv,dkv_tiles", [(1, 5000, 16, 2, 52), (3, 2727, 8, 2, 25), (1, 7000, 32, 4, 202)])
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
