"""Which candidate is quantized into which buffer and scored where, for grids of every size against the batch: LayerSearch on a
context that keeps track of them and computes nothing."""
import pytest
import torch

from paper_2309_15531_amd import binding as B
from paper_2309_15531_amd import search as S


class Tracker:
    """Stands in for a context: a buffer holds the (dimension, clip ratio) last quantized into it, a loss the candidate scored there."""

    def __init__(self):
        self.held, self.scored, self.allocated, self.launches, self.kept = {}, {}, 0, [], {}

    def alloc_score(self, rows, cols, device="cuda"):
        self.allocated += 1
        return torch.empty(8, dtype=torch.float16, device=device)

    def _put(self, dim, clip, dW, **kept):
        self.held[id(dW)] = (dim, clip)
        if kept:
            self.kept[(dim, clip)] = tuple(sorted((k, id(t)) for k, t in kept.items()))

    def adadim_quantize(self, W, dim, bits, group, clip=1.0, dW=None, dW_dtype=None, colscale=None, **kept):
        self._put(dim, clip, dW, **kept)

    adadim_quantize_meta16 = adadim_quantize

    def adadim_quantize_both(self, W, bits, group, colscale, oc, ic, clip=1.0, meta16=False):
        self._put(B.DIM_OC, clip, **oc)
        self._put(B.DIM_IC, clip, **ic)

    def adadim_layer_error_batch(self, dWs, dW_dtype, Hs, hmeta, losses, loss_rows=None, shape=None, at=None):
        self.launches.append(len(dWs))
        for i, t in zip(range(len(dWs)) if at is None else at, dWs):
            where = (losses.data_ptr() - self.base) // 4 + i
            assert where not in self.scored
            self.scored[where] = self.held[id(t)]

    def adadim_layer_error_batch_select(self, dWs, dW_dtype, Hs, hmeta, losses, best_dev, loss_rows=None, shape=None):
        self.adadim_layer_error_batch(dWs, dW_dtype, Hs, hmeta, losses)

    def adadim_select(self, losses, best_dev=None, to_host=True):
        assert len(self.scored) == losses.numel()


@pytest.mark.parametrize("meta16", [False, True])
@pytest.mark.parametrize("group,in_f", [(64, 256), (8, 40), (0, 256)])
@pytest.mark.parametrize("n_clips", [1, 2, 3, 4, 5, 9, 10, 20])
def test_every_candidate_is_scored_in_its_place_with_no_more_buffers_than_the_batch(n_clips, group, in_f, meta16):
    for batch in (1, 2, 3, 5, 7, 8, 100):
        for keep in (True, False):
            ctx, hp = Tracker(), type("Hp", (), {"colscale": None, "Hs": None, "hmeta": None})
            ls = S.LayerSearch(ctx, 128, in_f, 3, group, clips=S.clip_grid(n_clips), keep_winner=keep, batch=batch, device="cpu", meta16=meta16)
            n, most = 2 * n_clips, min(batch, 8)
            assert ctx.allocated <= most
            for select in (False, True):
                ctx.scored, ctx.launches, ctx.base = {}, [], ls.losses.data_ptr()
                ls.score_all(None, hp, select=select)
                assert [ctx.scored[i] for i in range(n)] == ls.cands
                assert len(ctx.launches) == -(-n // most), ctx.launches
            if keep and n <= most:
                assert len({v for v in ctx.kept.values()}) == n
                for k, cand in enumerate(ls.cands):
                    assert ("packed", id(ls._packed[k])) in ctx.kept[cand]
            else:
                assert not ctx.kept
