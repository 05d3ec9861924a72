"""Workspace sizes on both sides of the line from which the forward copies the
weight (no GPU needed)."""
import ctypes

import pytest

import paper_2505_17826_amd as R


@pytest.mark.parametrize("d,V", [(3584, 152064), (72, 1000)])
def test_step_workspace_has_room_for_the_weight_copy_only_where_it_is_made(d, V):
    """rft_ppo_clip_step copies the weight tile-blocked (Vpad x Kp bf16 values) for
    more than 10240 rows; up to there its workspace has no room for the copy."""
    L = R.lib()

    def size(f, T):
        tk = R.rft_tokens(T, 8, 0x1000, 0x1000, 0x1000)
        return f(R.RFT_OP_PPO_STEP, ctypes.byref(tk), d, V, R.RFT_BF16)

    copy = (V + 255) // 256 * 256 * ((d + 63) // 64 * 64) * 2
    # 256 rows on either side of the line: the per-row arrays grow by the same, up
    # to the rounding of each (about twenty) to 256 bytes
    for f in (L.rft_workspace_min_bytes, L.rft_workspace_bytes):
        below = size(f, 10240) - size(f, 10240 - 256)
        above = size(f, 10240 + 256) - size(f, 10240)
        assert abs(above - below - copy) <= 20 * 256, (above, below, copy)
