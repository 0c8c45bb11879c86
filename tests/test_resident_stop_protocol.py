"""How a resident tile's wavefronts agree to leave an abandoned launch, as a model
run through every interleaving on the host: in a half-sweep any wavefront may put
the sweep's number in the stop word (its wait has expired), all meet at a barrier,
and after a sweep's second half each then reads the word and leaves or goes on.  All
must leave after the same half-sweep."""
import pytest


def _leave_apart(numbered, waves, half_sweeps):
    """Whether some interleaving lets one wavefront leave after a half-sweep that another goes on from.  numbered: the
    word holds the sweep's number, otherwise only that some wavefront has set it.  A wavefront is (half-sweep, 0 at
    work / 1 at the barrier / 2 behind it), or its last half-sweep once it has left; the barrier opens when every
    wavefront that has not left is at it."""
    start = (((0, 0),) * waves, None)
    seen, todo = {start}, [start]
    while todo:
        ws, stop = todo.pop()
        left = [w for w in ws if isinstance(w, int)]
        live = [w for w in ws if not isinstance(w, int)]
        if left and (max(left) != min(left) or any(hs > min(left) for hs, _ in live)):
            return True
        nexts = []
        for i, w in enumerate(ws):
            if isinstance(w, int):
                continue
            hs, at = w
            if at == 0:
                nexts += [(ws[:i] + ((hs, 1),) + ws[i + 1:], s) for s in (stop, hs // 2)]
            elif at == 1 and all(x[1] == 1 for x in live):
                nexts.append((tuple(x if isinstance(x, int) else (x[0], 2) for x in ws), stop))
            elif at == 2:
                leaves = hs % 2 == 1 and (stop == hs // 2 if numbered else stop is not None)
                nexts.append((ws[:i] + (hs if leaves or hs + 1 == half_sweeps else (hs + 1, 0),) + ws[i + 1:], stop))
        for n in nexts:
            if n not in seen:
                seen.add(n)
                todo.append(n)
    return False


@pytest.mark.parametrize("waves", [2, 3])
def test_wavefronts_leave_together(waves):
    assert not _leave_apart(True, waves, 8)


def test_a_word_that_is_only_set_would_not_do():
    assert _leave_apart(False, 2, 6)
