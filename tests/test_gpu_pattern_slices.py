"""Pattern counts of longer captures, in chunks of 128 rows: both sides of every line between their kernels, ragged last
chunks, and the counts that the fused capture takes itself. Whole numbers, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2506_11104_amd import binding as B

pytestmark = pytest.mark.gpu
NAMES = ("vert_cnt", "diag_cnt", "vert_flag", "diag_flag")


def check_counts(mask, L, mu):
    """Counts and flags of a mask against those of its own true bits."""
    words = mask.true_bits.view(torch.uint8)  # [H][L][bytes], least significant bit first
    H = words.shape[0]
    for h in range(H):
        bits = ((words[h][:, :, None] >> torch.arange(8, device="cuda", dtype=torch.uint8)) & 1).reshape(L, -1)[:, :L].to(torch.int32)
        i = torch.arange(L, device="cuda")
        offset = (i[:, None] - i[None, :]).clamp_(min=0)
        vert = bits.sum(0, dtype=torch.int32)
        diag = torch.zeros(L, dtype=torch.int32, device="cuda").scatter_add_(0, offset.reshape(-1), bits.reshape(-1))
        size = (L - i).to(torch.float32)
        want = dict(vert_cnt=vert, diag_cnt=diag, vert_flag=vert.float() / size >= np.float32(mu), diag_flag=diag.float() / size >= np.float32(mu))
        assert int(bits.sum()) > 0
        for name in NAMES:
            assert torch.equal(getattr(mask, name)[h].to(want[name].dtype), want[name]), (h, name)


# both sides of the line at which captures are counted in chunks (832 tokens), 16 / 32 / 64 / 128 words
# per row, more than that (two waves per chunk: a last chunk of one row, one of 65, a whole one); a block index or none
@pytest.mark.parametrize("L,blocks", [(768, False), (769, False), (769, True), (832, False), (832, True), (833, False), (833, True), (1024, True), (1500, False), (1536, True), (1537, True), (2048, False),
                                      (1792, True), (1793, True), (1920, True), (2048, True), (2049, True),  # added up in the prep kernel, and by a launch
                                      (2049, False), (4096, False), (4097, False), (8192, False), (8193, False),
                                      (8257, False), (8320, True), (12300, False)])
def test_counts_in_chunks(L, blocks):
    gen = torch.Generator(device="cuda").manual_seed(L)
    A = torch.rand((2, L, L), generator=gen, device="cuda").tril_()
    A[1, L // 2:, 5] = 2.0
    A[1].diagonal(-3).fill_(2.0)
    m = B.build_mask(mode=B.DAM_FROM_ATTN_MAP, H=2, L=L, S=L + 70 if blocks else L, lam=0.5, eps=1e-8, tau=1.6, mu=0.4, attn_sum=A, blocks=blocks)
    check_counts(m, L, 0.4)


# a row tile per workgroup (whole rows: counted by the capture), several workgroups per row tile, short captures; more than 64
# words per row, which the waves of a workgroup hand each other behind barriers
@pytest.mark.parametrize("hq,hkv,L", [(64, 8, 1100), (32, 8, 2048), (64, 8, 1024), (16, 4, 1000), (128, 8, 700), (64, 8, 832), (64, 8, 833),
                                      (16, 4, 4100), (16, 8, 5000), (16, 4, 8192)])
def test_counts_of_a_fused_capture(hq, hkv, L):
    gen = torch.Generator(device="cuda").manual_seed(L)
    q, k = (torch.randn((h, L, 128), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hq, hkv))
    m = B.build_mask(mode=B.DAM_FROM_ATTN_MAP, H=hq, L=L, S=L, lam=0.5, eps=1e-8, tau=2.0 / np.sqrt(L), mu=0.3, qk=(q, k), blocks=False)
    check_counts(m, L, 0.3)
