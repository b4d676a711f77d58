"""Each branch of the kernels' dispatch at the sizes where it can go wrong: the edges of its tiles, remainders, the
smallest and largest of its range."""
import numpy as np
import pytest
import torch

import paper_2601_11822_amd as rs
import rs_synth as S
from oracle import lm
from tests.gpu_util import Rig, check_tensor, to_dev

pytestmark = pytest.mark.gpu
f32 = S.bf16_bits_to_f32


# rows and columns around the tiles of the head's passes: the weight-streaming one (up to 64 rows, 256 columns a
# workgroup), the 128-row and the 256-row tiles; every column count leaves a partly empty last tile
@pytest.mark.parametrize("shape,vocab,n", [(S.WIDE, 4228, 1), (S.WIDE, 4228, 64), (S.MID, 1028, 33), (S.MID, 1028, 65),
                                           (S.MID, 1284, 128), (S.MID, 2052, 129), (S.MID, 2052, 256), (S.MID, 1028, 300)])
def test_head_logits_and_choice(shape, vocab, n):
    rig = Rig(shape, n_blocks=4, max_prefill_tokens=16, max_decode_batch=n, max_context=64, with_oracle=False)
    try:
        hb = S.head_weights(shape.d_model, vocab)
        lm_head = hb["lm_head"].copy()
        lm_head[7] = lm_head[vocab - 3] = lm_head[vocab // 2]     # equal logits in three places: the lowest column wins
        hb["lm_head"] = lm_head
        hd = {k: to_dev(v) for k, v in hb.items()}
        rig.ctx.set_head(hd["embed"], hd["final_norm"], hd["lm_head"], vocab, -1)
        x_bits = S.hidden_states(n, shape.d_model, 9)
        row = n - 1                                               # ... and are this row's largest
        x_bits[row] = S.f32_to_bf16_bits(40.0 * f32(lm_head[7]))
        x = to_dev(x_bits)
        logits = torch.full((n, vocab), float("nan"), dtype=torch.float32, device="cuda")
        out, out2 = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        rig.ctx.lm_head_greedy(rs.RS_SIDE_DECODE, x, n, logits, out)
        rig.ctx.lm_head_greedy(rs.RS_SIDE_DECODE, x, n, None, out2)
        rig.ctx.sync(rs.RS_SIDE_DECODE)
        got, tok = logits.cpu().numpy(), out.cpu().numpy()
        check_tensor("logits", got, lm.head_logits(f32(x_bits), hb["final_norm"], lm_head, shape.rms_eps))
        assert np.array_equal(tok, np.argmax(got, axis=1)) and tok[row] == 7
        assert torch.equal(out, out2)
    finally:
        rig.close()
