"""The host's sizing of a plan (steps and kept pairs, counted run by run) against a key-by-key
statement of the same packing, and the radius tables' way into the descriptor."""
import numpy as np
import pytest

PATCH = 4


@pytest.fixture(scope="module")
def lv():
    import paper_2411_17178_amd as m
    m.load_library()
    return m


def _interval(n_q, n_k, c, r):
    ctr = ((2 * c + 1) * n_k) // (2 * n_q)
    return (0, n_k - 1) if r < 0 else (max(0, ctr - r), min(n_k - 1, ctr + r))


def _patches(side, band, nw, gh, gw):
    """(queries of the group, list of query lists) per group; window mode: (row, column) pairs."""
    if band:
        q = list(range(side * side))
        for a in range(0, len(q), 16 * nw):
            grp = q[a:a + 16 * nw]
            yield grp, [grp[i:i + 16] for i in range(0, len(grp), 16)]
        return
    for y0 in range(0, side, PATCH * gh):
        for x0 in range(0, side, PATCH * gw):
            ys, xs = range(y0, min(side, y0 + PATCH * gh)), range(x0, min(side, x0 + PATCH * gw))
            yield [(y, x) for y in ys for x in xs], \
                [[(y, x) for y in ys if (y - y0) // PATCH == a for x in xs if (x - x0) // PATCH == b]
                 for a in range(gh) for b in range(gw)]


def _count(scales, radius, qb, qe, band, nw, block_keys):
    steps = pairs = 0
    for k in range(qb, qe):
        sk = scales[k]
        parts = ([(0, min(k, 2))] + [(j, j) for j in range(3, k + 1)]) if band else [(j, j) for j in range(k + 1)]
        pps = (sk + 3) // 4
        shape = min(((-(-pps // h)) * (-(-pps // min(nw // h, pps))), h + min(nw // h, pps), -h, h)
                    for h in range(1, min(nw, pps) + 1))
        gh = shape[3]
        gw = min(nw // gh, pps)
        for queries, patches in _patches(sk, band, nw, gh, gw):
            keys = []                                       # the group's list: (part, y, x) or (part, column)
            keep = {}
            for p, (a, b) in enumerate(parts):
                n = sum(scales[j] ** 2 for j in range(a, b + 1)) if band else scales[b]
                rows = sk * sk if band else sk
                iv = {c: _interval(rows, n, c, radius) for c in (queries if band else range(sk))}
                keep[p] = iv
                if band:
                    keys += [(p, c) for c in range(iv[queries[0]][0], iv[queries[-1]][1] + 1)]
                else:
                    (ya, xa), (yb, xb) = queries[0], queries[-1]
                    keys += [(p, y, x) for y in range(iv[ya][0], iv[yb][1] + 1) for x in range(iv[xa][0], iv[xb][1] + 1)]
            for patch in patches:
                cnt, first = 0, 0
                for pos, key in enumerate(keys):
                    iv = keep[key[0]]
                    if band:
                        kept = sum(iv[q][0] <= key[1] <= iv[q][1] for q in patch)
                    else:
                        kept = sum(iv[y][0] <= key[1] <= iv[y][1] and iv[x][0] <= key[2] <= iv[x][1] for y, x in patch)
                    if not kept:
                        continue
                    pairs += kept
                    if cnt == 32 or (cnt and pos // block_keys - first > 1):
                        steps, cnt = steps + 1, 0
                    if cnt == 0:
                        first = pos // block_keys
                    cnt += 1
                steps += cnt > 0
    return steps, pairs


@pytest.mark.parametrize("waves,block_keys", [(4, 32), (8, 32), (16, 64)])
@pytest.mark.parametrize("band", [False, True])
@pytest.mark.parametrize("scales,radius,qs", [
    ((1, 2, 3, 4, 6, 9), 1, (0, 6)), ((2, 17), 0, (0, 2)),        # gaps between neighbouring queries' windows
    ((21, 3, 5), 0, (1, 3)), ((7, 2, 9, 4), -1, (0, 4)), ((1, 2, 13), 40, (2, 3)), ((5, 18), 2, (1, 2))])
def test_sizing_equals_the_key_by_key_count(lv, scales, radius, qs, band, waves, block_keys):
    st = lv.litevar_mask_plan_stats(scales, radius, None, 0, qs, waves_per_group=waves, mask_mode=int(band))
    assert (int(st.n_steps), int(st.retained_pairs)) == _count(scales, radius, *qs, band, waves, block_keys)


def test_radius_tables_of_every_number_type(lv):
    scales, table = (1, 2, 3), [[[1, 0, 0], [1, 2, 0], [2, 1, 3]]] * 2
    want = int(lv.litevar_mask_plan_stats(scales, 0, table).retained_pairs)
    for other in (np.array(table), np.array(table, dtype=np.float32), [[[float(v) for v in r] for r in t] for t in table],
                  [[tuple(str(v) for v in r) for r in t] for t in table]):
        assert int(lv.litevar_mask_plan_stats(scales, 0, other).retained_pairs) == want
    with pytest.raises(Exception):
        lv.litevar_mask_plan_stats(scales, 0, [[[-2, 0, 0], [1, 2, 0], [2, 1, 3]]])


def _wide_shape(side, h, w):
    """Rows and columns of a 32-query patch in groups of h x w patches of 16: the least sum of (rows + 6) (columns + 6)."""
    H, W = min(4 * h, side), min(4 * w, side)
    best = None
    for ph in range(1, min(H, 11) + 1):
        for pw in range(1, min(W, 32 // ph, 12 - ph) + 1):
            if -(-H // ph) * -(-W // pw) > 8:
                continue
            ny = side // H * -(-H // ph) + -(-(side % H) // ph)
            nx = side // W * -(-W // pw) + -(-(side % W) // pw)
            key = (ny * nx * (ph + 6) * (pw + 6) * 16 - pw, ph, pw)
            best = min(best or key, key)
    return best[1:]


def _dealt(lo, hi):
    """Rows lo .. hi dealt from four strips, the first of which are a row longer."""
    n = hi - lo + 1
    strips, at = [], lo
    for t in range(4):
        size = n // 4 + (t < n % 4)
        strips.append(range(at, at + size))
        at += size
    return [s[r] for r in range(n // 4 + 1) for s in strips if r < len(s)]


def _count_wide(scales, radius, qb, qe, band):
    steps = 0
    for k in range(qb, qe):
        sk = scales[k]
        parts = ([(0, min(k, 2))] + [(j, j) for j in range(3, k + 1)]) if band else [(j, j) for j in range(k + 1)]
        pps = (sk + 3) // 4
        gh = min(((-(-pps // h)) * (-(-pps // min(16 // h, pps))), h + min(16 // h, pps), -h, h) for h in range(1, min(16, pps) + 1))[3]
        gw = min(16 // gh, pps)
        if band:
            groups = [(list(range(a, min(sk * sk, a + 256))), None) for a in range(0, sk * sk, 256)]
            groups = [(q, [q[i:i + 32] for i in range(0, len(q), 32)]) for q, _ in groups]
        else:
            ph, pw = _wide_shape(sk, gh, gw)
            groups = []
            for y0 in range(0, sk, 4 * gh):
                for x0 in range(0, sk, 4 * gw):
                    ys, xs = list(range(y0, min(sk, y0 + 4 * gh))), list(range(x0, min(sk, x0 + 4 * gw)))
                    groups.append(([(y, x) for y in ys for x in xs],
                                   [(ys[a:a + ph], xs[b:b + pw]) for a in range(0, len(ys), ph) for b in range(0, len(xs), pw)]))
        for queries, patches in groups:
            keys, keep = [], {}
            for p, (a, b) in enumerate(parts):
                n = sum(scales[j] ** 2 for j in range(a, b + 1)) if band else scales[b]
                iv = {c: _interval(sk * sk if band else sk, n, c, radius) for c in (queries if band else range(sk))}
                keep[p] = iv
                if band:
                    keys += [(p, c) for c in range(iv[queries[0]][0], iv[queries[-1]][1] + 1)]
                    continue
                (ya, xa), (yb, xb) = queries[0], queries[-1]
                rows = (iv[ya][0], iv[yb][1])
                for y in (_dealt(*rows) if len(keys) >= 192 else range(rows[0], rows[1] + 1)):
                    keys += [(p, y, x) for x in range(iv[xa][0], iv[xb][1] + 1)]
            for patch in patches:
                cnt, first = 0, 0
                for pos, key in enumerate(keys):
                    iv = keep[key[0]]
                    if band:
                        kept = any(iv[q][0] <= key[1] <= iv[q][1] for q in patch)
                    else:
                        kept = any(iv[y][0] <= key[1] <= iv[y][1] for y in patch[0]) and any(iv[x][0] <= key[2] <= iv[x][1] for x in patch[1])
                    if not kept:
                        continue
                    if cnt == 32 or (cnt and pos // 64 - first > 1):
                        steps, cnt = steps + 1, 0
                    if cnt == 0:
                        first = pos // 64
                    cnt += 1
                steps += cnt > 0
    return steps


STEP_ADDR, STEP_MASK = 8, 9                      # sections of the blob


@pytest.mark.parametrize("band", [False, True])
@pytest.mark.parametrize("scales,radius,qs", [
    ((1, 2, 3, 4, 6, 9), 1, (0, 6)), ((2, 17), 0, (0, 2)), ((21, 3, 5), 0, (1, 3)), ((7, 2, 9, 4), -1, (0, 4)), ((1, 2, 13), 40, (2, 3)),
    ((5, 18), 2, (1, 2)), ((20, 12, 9), 0, (1, 3)), ((6, 10, 16, 23), 4, (2, 4)), ((30, 26), 3, (1, 2))])
def test_steps_of_the_wide_patches_equal_the_key_by_key_count(lv, scales, radius, qs, band):
    st = lv.litevar_mask_plan_stats(scales, radius, None, 0, qs, waves_per_group=16, mask_mode=int(band))
    want = _count_wide(scales, radius, *qs, band)
    assert int(st.off[STEP_MASK]) - int(st.off[STEP_ADDR]) == 1024 * want
