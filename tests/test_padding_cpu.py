"""The rows behind the tokens that weight-gradient products contract over: they count as cleared only once they are, also where a launch
fails, on a stand-in runtime without a GPU."""
import hip_standin as standin
import pytest

import synth_inputs as si


@pytest.mark.parametrize("layers,nth", [(2, 1), (12, 1), (12, 2)])  # the ranges of two layers are one launch, those of twelve two
def test_rows_whose_clearing_failed_are_cleared_by_the_next_product(tmp_path, layers, nth):
    model = si._gpt(layers, 72, 3, 200, 97, 64)
    script = """
rc, c = create(desc, 3)
assert rc == 0
out = []
for fail in (0, nth, 0, 0):
    S.standin_clear()
    S.standin_fail(b"zero_ranges", fail + 1 if fail else 0)  # behind the launch that clears the flags and vectors
    rc, why = hvp(c, 3, 64 if not out else 21)
    out.append([rc, why, sum("zero_ranges" in l[1] for l in log() if l[0] == "launch")])
show(out)
"""
    first, failed, again, third = standin.run(tmp_path, script, desc=standin.desc(model), nth=nth)
    chunks = 1 if layers == 2 else 2
    assert first[:2] == standin.ENQUEUED and first[2] == 1      # 192 tokens: nothing behind them
    assert failed[0] == -3 and failed[2] == nth
    assert again[:2] == standin.ENQUEUED and again[2] == 1 + chunks
    assert third[:2] == standin.ENQUEUED and third[2] == 1
