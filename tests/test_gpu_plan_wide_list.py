"""The work-list of the wide patches as the 32-query kernel reads it: the blob is copied to the host, every step's ring
offsets, mask bits and tokens are decoded, and the (query, key) pairs must be those of the oracle's mask, each once."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu
SEC_GROUPS, SEC_WAVES, SEC_PHASES, SEC_UNION, SEC_STEPS, RING = 4, 5, 6, 7, 8, 320
WIDE = (16, 0, 0, -1, 2)


def _piece(slot, piece):
    return slot * 128 + ((piece ^ ((slot ^ (slot >> 3)) & 7)) << 4)


def _words(blob, at, n, per):
    return blob[at:at + 4 * n * per].view(np.int32).reshape(n, per)


def _decode(plan, band, head):
    """The pairs as (query row, token) arrays; checks phases, padding and the three copies of a key's place on the way."""
    blob = plan.blob.cpu().numpy()
    off = [int(x) for x in plan.off]
    n_all, hg = int(plan.n_groups * plan.n_head_groups), int(plan.head_group[head]) if plan.n_heads else 0
    groups = _words(blob, off[SEC_GROUPS], n_all, 8)
    waves = _words(blob, off[SEC_WAVES] + n_all * 16 * 32, n_all * 8, 8)
    n_phases = int(plan.n_union_keys) // 64
    phases = _words(blob, off[SEC_PHASES], 1, 8 * n_phases)[0]
    union = _words(blob, off[SEC_UNION], 1, int(plan.n_union_keys))[0]
    rows, toks = [], []
    for G in range(hg * plan.n_groups, (hg + 1) * plan.n_groups):
        union_base, n_union, nph = int(groups[G, 0]), int(groups[G, 1]), int(groups[G, 2])
        for w in range(8):
            step0, n_steps, q_base, sk_ny, nx_kq, magic, valid, first_ends = (int(x) for x in waves[G * 8 + w])
            sk, ny, nx, valid = sk_ny & 0xffff, sk_ny >> 16, nx_kq & 0xffff, valid & 0xffffffff
            ends = phases[union_base // 64 * 8 + w * nph:][:nph]
            assert (np.diff(ends) >= 0).all() and ends[-1] == n_steps
            assert first_ends & 0xffffffff == int(ends[0]) | int(ends[min(2, nph - 1)]) << 16
            if not n_steps:
                continue
            steps = blob[off[SEC_STEPS] + step0 * 1024:][:n_steps * 1024].view(np.uint32).reshape(n_steps, 64, 4)
            n = np.arange(valid.bit_length())
            assert valid == (1 << len(n)) - 1 and nx > 0
            dy = n * magic >> 16
            assert (dy == n // nx).all() and (band or len(n) == ny * nx)
            row = q_base + dy * sk + (n - dy * nx)
            chunk_of = np.searchsorted(ends, np.arange(n_steps), side="right")          # in which the step ends
            lane = np.arange(64)
            for s in range(n_steps):
                d = steps[s]
                slot = (d[:32, 0] >> 7).astype(np.int64)
                assert (d[:, 0] == _piece(slot[lane & 31], lane >> 5)).all()
                v = np.stack([d[:, 1] & 0xffff, d[:, 1] >> 16, d[:, 2] & 0xffff, d[:, 2] >> 16])
                for i in range(4):
                    key = 8 * i + 4 * (lane >> 5) + ((lane & 15) >> 2)
                    assert (v[i] == _piece(slot[key], 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) + 8 * (lane & 1)).all()
                first = 64 * max(int(chunk_of[s]) - 1, 0)                               # the chunk before it may be read too
                upos = first + (slot - first) % RING
                assert (upos < 64 * (int(chunk_of[s]) + 1)).all()
                out = np.zeros((32, 32), bool)                                          # [dimension, key]
                for e in range(8):
                    for h in range(2):
                        word = d[32 * h:32 * h + 32, 3]
                        out[8 * h + e] = word >> (15 - 2 * (e >> 1) + 16 * (e & 1)) & 1
                        out[16 + 8 * h + e] = word >> (7 - 2 * (e >> 1) + 16 * (e & 1)) & 1
                assert not (d[:, 3] & 0x55005500 if not band else d[:, 3] & 0x55555555).any()   # (they would be exponent bits)
                kept = ~out[n] if band else ~out[dy] & ~out[ny + n - dy * nx]           # [query, key]
                assert (upos[kept.any(0)] < n_union).all()
                a, b = np.nonzero(kept)
                rows.append(row[a])
                toks.append(union[union_base + upos[b]])
    return np.concatenate(rows), np.concatenate(toks)


LISTS = [((1, 2, 3, 4, 5, 6, 7, 8), 1, None), ((9, 10, 11), 2, None), ((3, 13, 14), 0, (1, 3)), ((2, 17), 3, None), ((5, 19, 21), 2, (2, 3)),
         ((33, 7), 4, None), ((1, 3, 30), 40, None), ((12, 25), -1, (1, 2)), ((4, 9, 16), [2, 0, 5], None), ((20, 24), 5, (1, 2)),
         (workloads.configs.VAR256, 3, (9, 10)), (workloads.configs.VAR512, 4, (8, 10))]


@pytest.mark.parametrize("band", [False, True])
@pytest.mark.parametrize("scales,radius,q_scales", LISTS)
def test_pairs_of_the_wide_patches(scales, radius, q_scales, band):
    import paper_2411_17178_amd as lv
    radii = radius if isinstance(radius, list) else [radius] * len(scales)
    plan = lv.litevar_mask_build(scales, 0, radii, 1, q_scales, waves_per_group=WIDE, mask_mode=int(band))
    lv.litevar_plan_check(plan)
    _compare(plan, oracle.mask_dense(scales, radii, 1, q_scales, int(band)), band, 0)


def _compare(plan, want, band, head):
    rows, toks = _decode(plan, band, head)
    got = np.zeros(want.shape, np.int32)
    np.add.at(got, (rows, toks), 1)
    assert (got == want).all()
    kept = int(plan.retained_pairs_of_group[plan.head_group[head] if plan.n_heads else 0])
    assert len(rows) == kept == int(want.sum())


def test_pairs_of_the_patches_of_16_are_counted_by_their_walk():
    """The builder's own count of every patch, which it has compared with the host's."""
    import paper_2411_17178_amd as lv
    for waves, tables in ((16, 3), (16, 40), (8, 3), (8, 90), (4, 200)):        # with few and with many groups
        scales, K = (1, 3, 7, 13), 4
        rad = [[[h % 5, h // 5 % 7, h // 35, 1 + h % 2]] * K for h in range(tables)]
        plan = lv.litevar_mask_build(scales, 1, rad, 0, (3, 4), waves_per_group=waves)
        lv.litevar_plan_check(plan)
        n_all = int(plan.n_groups * plan.n_head_groups)
        w = _words(plan.blob.cpu().numpy(), int(plan.off[SEC_WAVES]), n_all * waves, 8)
        per_group = w[:, 5].reshape(plan.n_head_groups, -1).sum(1)
        assert per_group.tolist() == [int(x) for x in plan.retained_pairs_of_group[:plan.n_head_groups]]


@pytest.mark.parametrize("heads", [2, 40])       # few groups and many
def test_pairs_of_every_head_group(heads):
    import paper_2411_17178_amd as lv
    scales, K = (2, 5, 11, 18), 4
    tables = [[[h % 3, h // 3 % 4, h // 12, 1 + h % 4]] * K for h in range(heads)]
    plan = lv.litevar_mask_build(scales, 0, tables, 0, (2, 4), waves_per_group=WIDE)
    lv.litevar_plan_check(plan)
    for h in sorted({0, 1, heads // 2, heads - 1}):
        _compare(plan, oracle.mask_dense(scales, tables[h], 0, (2, 4)), False, h)


@pytest.mark.parametrize("waves", [4, 8, 16])
def test_patches_of_many_steps(waves):
    """More than 255 steps in a patch, whose counts travel in 32 bits."""
    import paper_2411_17178_amd as lv
    scales, tables = (96, 9), [[[-1, -1], [-1, h]] for h in range(5)]
    plan = lv.litevar_mask_build(scales, 0, tables, 0, (1, 2), waves_per_group=waves)
    lv.litevar_plan_check(plan)
    for h in (0, 4):
        want = oracle.mask_dense(scales, tables[h], 0, (1, 2))
        if waves == 16:
            _compare(plan, want, False, h)
        assert (lv.litevar_mask_export_dense(plan, head=h)[0].cpu().numpy() == want).all()
