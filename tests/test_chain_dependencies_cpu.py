"""What the entries of a chain laid out per XCD wait for (no GPU): every work item that wrote what an entry reads, or that still
reads or writes what the entry overwrites, is complete before it by what it waits for, directly or through others; and every
column, worked through in order, comes to its end.  Pixels are worked out here tap by tap."""
import numpy as np
import pytest

from paper_1901_00041_amd import st_conv as sc
from paper_1901_00041_amd import synth

ES = 2


def _network(batch, image, n_seq=8, blocks=9):
    """The first layers of every sequence's network on reused buffers, 1 GiB of address space per buffer."""
    ops, stage = [], 0
    steps = synth.resnet50_steps(batch, image)
    last = None
    for st in steps[:1 + 3 * blocks]:
        if last is not None and not (last.name.endswith("proj") and st.src == last.src):
            stage += 1
        last, s = st, st.shape
        for q in range(n_seq):
            buf = lambda i: ((q * 16 + i + 1) << 30) if i is not None else None
            epi = (sc.ST_EPI_RELU if st.relu else 0) | (sc.ST_EPI_RESIDUAL if st.res is not None else 0)
            w = ((n_seq * 16 + q) << 30) + st.index * (16 << 20)
            ops.append(sc.make_chain_op(sc.ST_OP_CONV, q, stage, sc.make_desc(s.N, s.C, s.H, s.W, s.K, s.R, s.S, s.stride, s.pad, "bf16", "bf16",
                                                                              buf(st.src), w, buf(st.dst), buf(st.res), epi)))
            if st.pool_after:
                d = sc.make_desc(s.N, s.K, s.P, s.Q, s.K, 3, 3, 2, 1, "bf16", "bf16", buf(st.dst), None, buf(st.pool_dst))
                ops.append(sc.make_chain_op(sc.ST_OP_MAXPOOL, q, stage + 1, d))
        if st.pool_after:
            stage += 1
    return ops


def _out_size(d):
    return (d.H + 2 * d.pad - d.R) // d.stride + 1, (d.W + 2 * d.pad - d.S) // d.stride + 1


def _written(op, info, tile_m):
    """Output pixels of one tile index, as an array of linear indices."""
    d = op.conv
    P, Q = _out_size(d)
    if op.kind == sc.ST_OP_MAXPOOL:
        v = np.arange(tile_m * 256, min((tile_m + 1) * 256, d.N * P * Q * (d.C // 8)))
        return np.unique(v // (d.C // 8))
    t = info.tile
    if t.row_tiled:
        qt, pg = -(-Q // 128), -(-P // t.rows_per_tile)
        g, seg = divmod(tile_m, qt)
        n, p = g // pg, (g % pg) * t.rows_per_tile
        q = np.arange(seg * 128, min(Q, seg * 128 + 128))
        return np.concatenate([(n * P + r) * Q + q for r in range(p, min(P, p + t.rows_per_tile))])
    return np.arange(tile_m * t.MT, min((tile_m + 1) * t.MT, d.N * P * Q))


def _read(op, pixels):
    d = op.conv
    P, Q = _out_size(d)
    n, p, q = pixels // (P * Q), pixels % (P * Q) // Q, pixels % Q
    out = []
    for r in range(d.R):
        for s in range(d.S):
            h, w = p * d.stride - d.pad + r, q * d.stride - d.pad + s
            ok = (h >= 0) & (h < d.H) & (w >= 0) & (w < d.W)
            out.append(((n * d.H + h) * d.W + w)[ok])
    return np.unique(np.concatenate(out)) if out else np.zeros(0, int)


def _check(ops, chain, sequence):
    items, deps, cols = chain.worklist(), chain.dependencies().astype(np.int64), chain.columns().astype(np.int64)
    assert len(deps) == len(items) and sorted(deps[:, 0]) == list(range(len(items)))
    infos = [chain.op_info(i) for i in range(len(ops))]
    entry_of_flag = np.argsort(deps[:, 0])
    mine = [e for e in entry_of_flag if ops[items["tenant"][e]].sequence == sequence]       # by flag: stage by stage
    index = {int(deps[e, 0]): k for k, e in enumerate(mine)}
    # complete[k]: bit set of the sequence's entries known to be complete when entry k starts
    complete = []
    for e in mine:
        known = 0
        for b, c in ((deps[e, 1], deps[e, 2]), (deps[e, 3], deps[e, 4])):
            for f in range(b, b + c):
                known |= (1 << index[f]) | complete[index[f]]
        complete.append(known)
    of_op = {}
    for k, e in enumerate(mine):
        of_op.setdefault(int(items["tenant"][e]), []).append((k, int(items["tile_m"][e])))
    mask = {i: sum(1 << k for k, _ in v) for i, v in of_op.items()}
    order = sorted(of_op, key=lambda i: ops[i].stage)
    waits_by_tile = 0
    for i in order:
        T = ops[i].conv
        earlier = [j for j in order if ops[j].stage < ops[i].stage]
        writers = [j for j in earlier if ops[j].conv.y == T.x]
        producer = writers[-1] if writers else None
        whole = 0
        for j in earlier:
            U = ops[j].conv
            reads_u = [U.x] + ([U.residual] if U.epilogue & sc.ST_EPI_RESIDUAL else [])
            if T.y in reads_u + [U.y] or (T.epilogue & sc.ST_EPI_RESIDUAL and T.residual == U.y) or (T.x == U.y and j != producer):
                whole |= mask[j]
        if producer is not None:
            writes = [(1 << k, set(_written(ops[producer], infos[producer], m).tolist())) for k, m in of_op[producer]]
        by_tile = {}
        for k, m in of_op[i]:
            assert whole & ~complete[k] == 0, (i, m)
            if producer is None:
                continue
            if m not in by_tile:
                need = set(_read(ops[i], _written(ops[i], infos[i], m)).tolist())
                by_tile[m] = sum(bit for bit, px in writes if px & need)
            assert by_tile[m] & ~complete[k] == 0, (i, m)
            waits_by_tile += int(mask[producer] & ~complete[k] != 0)
    # the columns come to their end
    done, at = set(), list(cols[:-1])
    moved = True
    while moved:
        moved = False
        for j in range(len(at)):
            while at[j] < cols[j + 1] and all(f in done for b, c in ((deps[at[j], 1], deps[at[j], 2]), (deps[at[j], 3], deps[at[j], 4])) for f in range(b, b + c)):
                done.add(int(deps[at[j], 0]))
                at[j] += 1
                moved = True
    assert len(done) == len(items)
    return waits_by_tile


@pytest.mark.parametrize("batch,image,opts", [(2, 64, {}), (1, 96, {}), (3, 56, {"tile_cfg": 5}), (2, 48, {"tile_cfg": 4, "split_k": 2}), (1, 64, {"tile_cfg": 6, "split_k": 3}),
                                              (1, 80, {"tile_cfg": 1}), (2, 40, {"target_items": 300})])
def test_every_entry_waits_for_what_it_touches(batch, image, opts):
    ops = _network(batch, image)
    chain = sc.Chain(ops, sc.plan_opts(host_only=1, **opts))
    assert chain.info().n_queues == 8
    assert _check(ops, chain, 0) > 0 or opts.get("split_k", 1) > 1       # (neighbouring split-K stages share a workspace: in order)


def _layer(C, side, K, window, pad, x, y, stride=1, n=2, res=None, w=1 << 40):
    epi = sc.ST_EPI_RESIDUAL if res is not None else 0
    return sc.make_desc(n, C, side, side, K, window, window, stride, pad, "bf16", "bf16", x, w, y, res, epi)


@pytest.mark.parametrize("second,tile_by_tile", [
    (_layer(64, 28, 64, 3, 1, 2 << 30, 3 << 30), True),
    (_layer(64, 28, 64, 1, 0, 2 << 30, 3 << 30, res=4 << 30), True),
    (_layer(64, 28, 64, 3, 1, 2 << 30, 1 << 30), False),                        # overwrites what the first still reads
    (_layer(64, 28, 64, 1, 0, 2 << 30, 3 << 30, res=2 << 30), False),           # the residual is the first's output too
    (_layer(64, 28, 64, 3, 1, (2 << 30) + 128, 3 << 30), False),                # shifted
    (_layer(32, 28, 64, 3, 1, 2 << 30, 3 << 30), False),                        # half of the bytes, other channels
    (_layer(64, 14, 64, 3, 1, 2 << 30, 3 << 30, n=8), False),                   # the same bytes, another shape
    (_layer(64, 28, 64, 1, 0, 2 << 30, 3 << 30, stride=30), False),             # reads one pixel: the rest would be waited for by nobody
    (_layer(64, 28, 64, 3, 1, 5 << 30, 3 << 30), False),                        # does not read the first at all
    (_layer(64, 28, 64, 3, 1, 2 << 30, 1 << 40, w=2 << 40), False),                        # overwrites the first's filters
])
def test_which_layers_wait_tile_by_tile(second, tile_by_tile):
    first = _layer(64, 28, 64, 3, 1, 1 << 30, 2 << 30)
    third = _layer(64, second.H, 64, 1, 0, 3 << 30, 6 << 30)
    ops = [sc.make_chain_op(sc.ST_OP_CONV, 0, s, d) for s, d in enumerate((first, second, third))]
    chain = sc.Chain(ops, sc.plan_opts(host_only=1, chain_queues=2, tile_cfg=4))
    deps, items = chain.dependencies(), chain.worklist()
    mine = deps[items["tenant"] == 1]
    first_count = int((items["tenant"] == 0).sum())
    assert (mine[:, 4] > 0).all() if tile_by_tile else (mine[:, 4] == 0).all()
    assert (mine[:, 2] == (0 if tile_by_tile else first_count)).all()
