"""The adjoints' buffers of layers whose weight-gradient products wait are memory that a context can do without: it is made without them where
room is scarce, and gives them up for the vector of a Hessian column.  On a stand-in runtime without a GPU."""
import hip_standin as standin

import synth_inputs as si

MODEL = si._gpt(6, 264, 3, 1048, 97, 77)  # buffers for four layers

SIZES = """
rc, c = create(desc, 4)
assert rc == 0
whole = S.standin_used()
assert whole == L.hf_workspace_bytes(c)
n = L.hf_num_params(c)
L.hf_destroy(c)
assert S.standin_used() == 0
S.standin_limit(whole - 1)
rc, c = create(desc, 4)
assert rc == 0
least = S.standin_used()
assert least == L.hf_workspace_bytes(c) and least < whole
"""


def test_a_context_that_fits_only_without_them(tmp_path):
    got = standin.run(tmp_path, SIZES + """
a = hvp(c, 4, 77)
L.hf_destroy(c)
b = S.standin_used()
S.standin_limit(least - 1)
rc, c = create(desc, 4)
show([a, b, rc, L.hf_last_error(None).decode()])
""", desc=standin.desc(MODEL))
    assert got[0] == standin.ENQUEUED and got[1] == 0
    assert got[2] == -2 and "hipMalloc" in got[3]


def test_room_that_is_gone_when_it_is_asked_for(tmp_path):
    got = standin.run(tmp_path, SIZES + """
L.hf_destroy(c)
log()
S.standin_free(1 << 40)
rc, c = create(desc, 4)
tried = [l[0] for l in log()]
pending = S.hipGetLastError()
show([rc, tried, pending, S.standin_used() == least == L.hf_workspace_bytes(c), hvp(c, 4, 77)])
""", desc=standin.desc(MODEL))
    assert got == [0, ["malloc", "refused"], 0, True, standin.ENQUEUED]


def test_they_leave_an_eighth_of_the_card(tmp_path):
    got = standin.run(tmp_path, SIZES + """
L.hf_destroy(c)
out = []
for room in (whole * 8 // 7 - 256, whole * 8 // 7 + 256):
    S.standin_limit(room)
    rc, c = create(desc, 4)
    out.append([rc, S.standin_used()])
    L.hf_destroy(c)
show([least, whole, out])
""", desc=standin.desc(MODEL))
    least, whole, out = got
    assert out == [[0, least], [0, whole]]


def test_a_column_that_fits_only_without_them(tmp_path):
    got = standin.run(tmp_path, SIZES + """
L.hf_destroy(c)
S.standin_limit(1 << 60)
rc, c = create(desc, 4)          # with them
first = hvp(c, 4, 77)
S.standin_limit(max(whole, least + n * 4))  # what the rest of the program leaves
a = [L.hf_hessian_column(c, P, X, Y, 4, 77, 5, OUT, None, None), L.hf_last_error(c).decode()]
again = hvp(c, 4, 77)
used = S.standin_used() - n * 4
b = L.hf_workspace_bytes(c)
L.hf_destroy(c)
show([first, a, again, used == b == least, S.standin_used()])
""", desc=standin.desc(MODEL))
    assert got == [standin.ENQUEUED] * 3 + [True, 0]


def test_widths_that_no_common_launch_takes_have_none(tmp_path):
    bytes_of = lambda model: standin.run(tmp_path, "rc, c = create(desc, 4)\nshow([rc, len([l for l in log() if l[0] == 'malloc'])])", desc=standin.desc(model))
    assert bytes_of(MODEL) == [0, 2]
    assert bytes_of(si._gpt(6, 260, 4, 1040, 97, 77)) == [0, 1]
    assert bytes_of(si._gpt(6, 264, 3, 1044, 97, 77)) == [0, 1]
