"""Host replay of the weight gradient's copies ahead (no GPU).

k_wgrad_tr's four copying waves run up to `ahead` bricks in front of the
products over a ring of 6 + 4 ahead halo plane slots and ahead + 1
output-gradient buffers, and wait only until as many of their copies are
outstanding as the later bricks have at least.  This test transcribes that
schedule and holds it against the plain rule: when a brick is multiplied, its
six planes and its output gradient are complete in the slots the products
read, and no copy in flight writes to one of them."""
import pytest


def replay(G, per, RS, n):
    ahead = 4 if RS == 1 else 3
    ring = 6 + 4 * ahead
    nbx, nby, nbz = G >> 4, G >> 2, G >> 2
    nbricks = n * nbz * nby * nbx
    dy_items = 16 * (40 if RS == 1 else 66)
    dy_copies = (dy_items + 63) // 64
    deepest = 0
    for b0 in range(0, nbricks, per):
        b1 = min(b0 + per, nbricks)

        def follows(b):
            return b > b0 and b % nbz != 0

        queue = [[] for _ in range(4)]      # copies in order, by wave: (target, content)
        planes, bufs = {}, {}               # landed pieces by target
        nxt, end, wslot, wbuf, base = b0, 0, 0, 0, 0
        bslot, bbuf = 0, 0

        def land(w, keep):
            while len(queue[w]) > keep:
                (where, at, piece), what = queue[w].pop(0)
                (planes if where == "p" else bufs).setdefault(at, {})[piece] = what

        def fill(b):
            nonlocal nxt, end, wslot, wbuf
            while nxt < b1 and nxt - b <= ahead:
                f = follows(nxt)
                count = 4 if f else 6
                if end + count - base > ring:
                    break
                for p in range(2 if f else 0, 6):
                    at = (wslot + p - (2 if f else 0)) % ring
                    z = (nxt // nbz, (nxt % nbz) * 4 - 1 + p)
                    for w in range(2):
                        for i in range(2):
                            queue[w].append((("p", at, 2 * w + i), z))
                for c in range(dy_copies):
                    queue[2 + c % 2].append((("d", wbuf, c), nxt))
                end += count
                wslot = (wslot + count) % ring
                wbuf = 0 if wbuf == ahead else wbuf + 1
                nxt += 1

        for b in range(b0, b1):
            if b == b0:
                fill(b)
            later = min(nxt - b - 1, 4)
            assert later >= 0, "the brick's copies were issued"
            deepest = max(deepest, later)
            for w in range(4):
                allowed = later * (8 if w < 2 else dy_copies // 2)
                assert allowed < 64
                land(w, allowed)
            if b > b0:
                fill(b)
            mine = [(bslot + p) % ring for p in range(6)]
            for p, at in enumerate(mine):
                z = (b // nbz, (b % nbz) * 4 - 1 + p)
                assert planes[at] == {k: z for k in range(4)}, (b, p)
            assert bufs[bbuf] == {c: b for c in range(dy_copies)}, b
            for q in queue:
                for (where, at, _), _what in q:
                    assert at not in mine if where == "p" else at != bbuf, b
            step = 4 if follows(b + 1) else 6
            base += step
            bslot = (bslot + step) % ring
            bbuf = 0 if bbuf == ahead else bbuf + 1
    return deepest


@pytest.mark.parametrize("RS", [1, 2])
@pytest.mark.parametrize("G,per,n", [(16, 1, 2), (16, 2, 2), (16, 3, 3), (16, 16, 5), (32, 7, 1), (32, 21, 2),
                                     (64, 63, 1)])
def test_copies_ahead_land_in_free_slots(G, per, n, RS):
    deepest = replay(G, per, RS, n)
    assert deepest >= min(per - 1, 2)
