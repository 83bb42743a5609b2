"""Gradients of the two vocabulary tables and the position table inside a whole training step, row by row: token ids as text has them
give rows that are orders of magnitude apart, and a norm over the table would see the few frequent ones only."""
import pytest
import torch

from paper_2511_11641_amd import binding as B
from paper_2511_11641_amd.stack import DecoderStack

pytestmark = pytest.mark.gpu

LLAMA = {"d": 2048, "h": 32, "h_kv": 32, "d_h": 64, "d_ff": 5461, "gated": True, "rope": True, "bias": False, "causal": True}
GPT2 = {"d": 1024, "h": 16, "h_kv": 16, "d_h": 64, "d_ff": 4096, "gated": False, "rope": False, "bias": True, "causal": True}


@pytest.mark.parametrize("cfg,vocab,Bsz,L", [(LLAMA, 32000, 32, 256), (GPT2, 50304, 3, 381)], ids=["llama", "gpt2"])
def test_table_gradients_row_by_row(cfg, vocab, Bsz, L):
    st = DecoderStack(B.Context("cuda:0"), dict(cfg, B=Bsz, L=L), 1, vocab, keep=(1, 2), seed=4, train=True)
    gen = torch.Generator(device="cuda").manual_seed(6)
    ids = (vocab * torch.rand(Bsz * L + 1, device="cuda", generator=gen) ** 3).long().clamp_(max=vocab - 1)
    ids, targets = ids[:-1].contiguous(), ids[1:].contiguous()
    st.train_step(ids, targets)
    # what the step leaves behind: the gradient of the logits in their buffer, the final hidden rows, the gradient at the embedding
    dl, hf, dx = st.logits.double(), st.hf.double(), st.dxa.double()

    def rows_close(got, want, what):
        # a bf16 result is at most 2^-9 off its value, element by element; fp32 sums of bf16 products add well below that
        err, ref = (got.double() - want).norm(dim=1), want.norm(dim=1)
        assert float(ref.max()) > 0 and bool((err <= 2.0 ** -8 * ref + 1e-7 * ref.max()).all()), f"{what}: row {int((err / (ref + 1e-30)).argmax())}"

    rows_close(st.lm.g, dl.t().contiguous() @ hf, "projection")
    want = torch.zeros((vocab, cfg["d"]), dtype=torch.float64, device="cuda").index_add_(0, ids, dx)
    rows_close(st.emb.g, want, "embedding")
    seen = torch.zeros(vocab, dtype=torch.bool, device="cuda").index_fill_(0, ids, True)
    assert not st.emb.g[~seen].any() and bool(st.emb.g[seen].any(dim=1).all())
    if st.pos is not None:
        rows_close(st.pos.g, dx.reshape(Bsz, L, -1).sum(dim=0), "position")
