"""GPU: the pair-hub tables from narrow membership rows (a row is narrowed where
memory is short): lane groups share a row, and there are more panels."""

import numpy as np
import pytest

import oracle
import synth
from oracle.pattern import compile_pattern
from test_gpu_pair_tables import _hub_graph

pytestmark = pytest.mark.gpu

A = pytest.importorskip("paper_2601_01388_amd")


# panels of 32 hubs a word: several at most widths, the last one partly filled
@pytest.mark.parametrize("words", [1, 2, 4, 16])
@pytest.mark.parametrize("hubs", [129, 2300])
def test_narrow_rows_against_oracle(words, hubs):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01388_amd.session import Session
    s = Session(0)
    assert A.lib().agis_internal_row_words(s.ctx, words) == A.AGIS_OK
    g = _hub_graph(hubs, 6 * hubs + 200, seed=hubs)
    G = s.graph(g.off, g.nbr)
    T = s.tables(G, cv_seed=1)
    OT = oracle.Tables(g, cv_seed=1)
    idx = np.arange(1000, dtype=np.uint64)
    for name in ("4-cycle", "house", "4-clique"):
        p = synth.named_pattern(name)
        for mode in ("switch", "uniform"):
            ref = oracle.Sampler(g, OT, compile_pattern(p.k, p.edges, mode=mode), seed=5).records(idx)
            got = s.dump(G, T, p, 5, idx, mode=mode, rowtab="on")
            for f in ("v", "num", "den", "x", "steps", "fail_step"):
                assert np.array_equal(got[f], ref[f]), (hubs, words, name, mode, f)
    T.close()
    G.close()
    s.close()
