"""The lanes engine's event loop where its windows, bytes and bounds end.

Thresholds of every width the engine takes (1 to 32 planes: each number of
Philox quads, whole and partial), windows of 32 events cut at every kind of
place (ragged words, staggered replicas, launches of a few events, runs that
cross a multiple of 2^32), states of weight zero, and totals that grow past
the window's bound.  Exact against the oracle.
"""

import numpy as np
import pytest

import paper_2412_16613_amd as bwg
from oracle import ssa
from workloads import (frank_network, open_network, paper_network, random_network,
                       random_wide_network)
from workloads.frank import (_A_TO_D, _A_TO_L, _AD_TO_2D, _AL_TO_2L, _LD_TO_2A, _net)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def exact_network(n_tot, cu, ca, ci):
    """Frank network with integer weights; 0 leaves the reactions out."""
    rx = [(_A_TO_L, cu), (_A_TO_D, cu), (_AL_TO_2L, ca), (_AD_TO_2D, ca), (_LD_TO_2A, ci)]
    rx = [r for r in rx if r[1]]
    return _net([r[0] for r in rx], [r[1] for r in rx], n_tot, exact_integer=True)


def check(torch, net, M, init, ops, seed=3, **kw):
    print("case", net["n_tot"], net["rates"], M, init, ops, flush=True)
    e = bwg.Ensemble(bwg.Network(net), M, seed=seed, net_id=5, engine="lanes", **kw)
    o = ssa.OracleEnsemble(net, M, seed=seed, net_id=5)
    e.init(init)
    o.init(init)
    for op, v in ops:
        getattr(e, op)(v)
        getattr(o, op)(v)
    np.testing.assert_array_equal(e.read_counts().cpu().numpy(), o.counts)
    ev, real = e.read_events()
    np.testing.assert_array_equal(ev.cpu().numpy().astype(np.uint64), o.E)
    want = np.zeros((M + 31) // 32, np.uint64)
    np.add.at(want, np.arange(M) // 32, o.real.astype(np.uint64))
    np.testing.assert_array_equal(real.cpu().numpy().astype(np.uint64), want)


# n_tot of the paper's network by threshold planes 1 .. 20
PAPER_N = {1: 2, 2: 3, 3: 4, 4: 6, 5: 8, 6: 11, 7: 16, 8: 20, 9: 32, 10: 40, 11: 60, 12: 90,
           13: 120, 14: 180, 15: 250, 16: 360, 17: 500, 18: 700, 19: 1000, 20: 1400}


@pytest.mark.parametrize("B", sorted(PAPER_N))
def test_every_width_of_small_weights(torch, B):
    net = paper_network(PAPER_N[B])
    assert bwg.Network(net).quantized()["B"] == B
    check(torch, net, 97, ("multinomial",), [("step", 333)])


@pytest.mark.parametrize("B,n_tot,cu,ca,ci", [
    (21, 1000, 100, 4, 4), (22, 1000, 900, 8, 8), (23, 1024, 164, 16, 16), (24, 3535, 177, 2, 2),
    (25, 4000, 300, 4, 4), (26, 1000, 25000, 8, 8), (27, 1000, 20000, 256, 256),
    (28, 1000, 70000, 512, 512), (29, 1000, 65535, 1024, 1024), (30, 1000, 65536, 2048, 2048),
    (31, 1000, 131072, 4096, 4096), (32, 1000, 1 << 19, 8192, 8192),
    (32, 12, 1 << 27, 1 << 24, 1 << 24)])
def test_every_width_of_large_weights(torch, B, n_tot, cu, ca, ci):
    net = exact_network(n_tot, cu, ca, ci)
    assert bwg.Network(net).quantized()["B"] == B
    check(torch, net, 65, ("fixed", (n_tot // 4, n_tot // 5, n_tot - n_tot // 4 - n_tot // 5)),
          [("step", 500)])


# planes on both sides of the rule's quads; the cases above run in pairs of waves
@pytest.mark.parametrize("words", [511, 512, 513, 2048, 2049])
@pytest.mark.parametrize("n_tot,cu,ca,ci", [(6, 1, 1, 1), (200, 50, 4, 4), (1000, 100, 4, 4),
                                            (1000, 1 << 19, 8192, 8192)],
                         ids=["few", "B17", "B21", "B32"])
def test_one_wave_and_pairs_of_waves(torch, n_tot, cu, ca, ci, words):
    """Windows that end within a launch, replicas that end early and words of
    one half wave only, on both sides of the sizes where a second wave draws."""
    net = exact_network(n_tot, cu, ca, ci)
    check(torch, net, 32 * words - 31, ("fixed", (0, 0, n_tot)),
          [("step", 33), ("advance", 60 / bwg.Network(net).quantized()["Lambda"]), ("step", 100)])


@pytest.mark.parametrize("n_tot", [5, 40])
def test_pairs_of_waves_that_end_early(torch, n_tot):
    check(torch, frank_network(n_tot, k0=0.3), 64 * 40 + 7, ("fixed", (0, 0, n_tot)),
          [("step", 40 * n_tot), ("step", 3000)])


@pytest.mark.parametrize("steps", [31, 32, 33, 64, 65, 96, 97, 160, 1000])
def test_pairs_of_waves_leave_at_the_same_window(torch, steps):
    """One pair of waves whose chain ends in the first, an even or an odd, the
    last or no window of a launch, by the seed; a second launch finds it ended."""
    for seed in range(8):
        check(torch, paper_network(3), 64, ("multinomial",), [("step", steps), ("step", steps)],
              seed=seed)


@pytest.mark.parametrize("cu,ca,ci", [(7, 0, 0), (0, 4, 0), (0, 0, 2), (5, 8, 0), (70000, 0, 64)])
def test_absent_reactions(torch, cu, ca, ci):
    net = exact_network(90, cu, ca, ci)
    check(torch, net, 130, ("fixed", (30, 25, 35)), [("step", 700)])


@pytest.mark.parametrize("M", [1, 31, 32, 33, 64, 65, 255, 257])
def test_ragged_words_and_staggered_replicas(torch, M):
    check(torch, frank_network(50, k0=0.04), M, ("fixed", (0, 0, 50)),
          [("advance", 1.0), ("step", 1), ("step", 31), ("advance", 3.0), ("step", 64)])


@pytest.mark.parametrize("epl", [1, 31, 32, 33, 100])
def test_launches_of_few_events(torch, epl):
    check(torch, frank_network(64), 70, ("fixed", (0, 0, 64)), [("advance", 2.0), ("step", 90)],
          events_per_launch=epl)


def test_totals_that_outgrow_the_bound(torch):
    # one L among A: the total climbs from almost nothing to its largest
    # value within a few events, window after window
    net = exact_network(200, 0, 64, 64)
    check(torch, net, 333, ("fixed", (1, 0, 199)), [("step", 2000)])
    # and a state that nothing leaves
    check(torch, net, 40, ("fixed", (200, 0, 0)), [("step", 100)])


@pytest.mark.parametrize("start", [(1 << 26) - 77, (1 << 32) - 200, (1 << 34) - 31])
def test_event_indices_cross_a_high_bit(torch, start):
    net = frank_network(40, k0=0.05)
    M = 77
    e = bwg.Ensemble(bwg.Network(net), M, seed=8, net_id=1, engine="lanes")
    o = ssa.OracleEnsemble(net, M, seed=8, net_id=1)
    e.init_fixed((0, 0, 40))
    o.init(("fixed", (0, 0, 40)))
    e.advance(1.0)
    o.advance(1.0)
    # the same chain with every event index moved up (regions 3 and 4 of a
    # checkpoint hold the events run and to reach)
    blob = bytearray(e.save())
    h = np.frombuffer(blob, dtype=np.uint64, count=32)
    for k in range(int(h[11])):
        if int(h[12 + 3 * k]) in (3, 4):
            np.frombuffer(blob, dtype=np.uint64, count=int(h[14 + 3 * k]) // 8,
                          offset=int(h[13 + 3 * k]))[:M] += np.uint64(start)
    e.restore(bytes(blob))
    o.E = o.E + np.uint64(start)
    e.step(500)
    o.step(500)
    np.testing.assert_array_equal(e.read_counts().cpu().numpy(), o.counts)
    np.testing.assert_array_equal(e.read_events()[0].cpu().numpy().astype(np.uint64), o.E)


@pytest.mark.parametrize("net", [frank_network(32), frank_network(61, k0=0.02)],
                         ids=["precompiled", "compiled"])
def test_word_events_cross_a_high_bit(torch, net):
    """The same for the word kernel of large ensembles, against the lanes
    loop: lanes that reach the crossing at different events of a launch, some
    of which do not reach it."""
    M = 32 * 32768 + 45
    n = bwg.Network(net)
    got = []
    for engine in ("bitwise", "lanes"):
        e = bwg.Ensemble(n, M, seed=8, net_id=1, engine=engine)
        e.init_fixed((0, 0, net["n_tot"]))
        e.advance(0.2)
        blob = bytearray(e.save())
        h = np.frombuffer(blob, dtype=np.uint64, count=32)
        for k in range(int(h[11])):
            if int(h[12 + 3 * k]) in (3, 4):
                v = np.frombuffer(blob, dtype=np.uint64, count=int(h[14 + 3 * k]) // 8,
                                  offset=int(h[13 + 3 * k]))
                v[:M] += np.uint64((1 << 32) - 200)
        e.restore(bytes(blob))
        e.step(180)
        e.step(300)
        got.append((e.read_counts().cpu().numpy(), e.read_events()[0].cpu().numpy()))
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])
    assert (got[0][1].astype(np.uint64) >= 1 << 32).all()


# ---- which loop a bit-sliced ensemble runs --------------------------------------

@pytest.mark.parametrize("net,init", [
    (frank_network(32), ("fixed", (0, 0, 32))),                 # precompiled weights
    (frank_network(1024), ("fixed", (0, 0, 1024))),
    (frank_network(100, k0=0.03), ("fixed", (0, 0, 100))),      # compiled for the network
    (paper_network(64), ("multinomial",)),
], ids=["frank32", "frank1024", "frank100", "paper64"])
def test_word_kernels_of_small_ensembles(torch, net, init):
    """A word width asked for keeps the word kernels, which small ensembles
    no longer run by default."""
    M = 4096 + 77
    e = bwg.Ensemble(bwg.Network(net), M, seed=6, net_id=2, word_bits=32)
    o = ssa.OracleEnsemble(net, M, seed=6, net_id=2)
    e.init(init)
    o.init(init)
    for t in (0.2, 0.9):
        e.advance(t)
        o.advance(t)
    e.step(60)
    o.step(60)
    np.testing.assert_array_equal(e.read_counts().cpu().numpy(), o.counts)
    np.testing.assert_array_equal(e.read_events()[0].cpu().numpy().astype(np.uint64), o.E)


@pytest.mark.parametrize("n_tot,words", [(32, 16384), (100, 20480), (32, 24576), (200, 24576),
                                         (1024, 49152)])
@pytest.mark.parametrize("more", [0, 1])
def test_both_sides_of_the_size_rule(torch, n_tot, words, more):
    """Around the size at which the default leaves the lanes loop, every
    choice gives the same state."""
    M = 32 * words + more
    net = bwg.Network(frank_network(n_tot))
    got = []
    for kw in (dict(), dict(word_bits=32), dict(engine="lanes")):
        e = bwg.Ensemble(net, M, seed=2, **kw)
        e.init_fixed((0, 0, n_tot)).advance(0.2).step(40)
        got.append((e.read_counts(), *e.read_events()))
    for g in got[1:]:
        for x, y in zip(g, got[0]):
            assert bool((x == y).all())


def active_ms(torch, net, M, start, events, **kw):
    e = bwg.Ensemble(net, M, seed=3, **kw)
    ms = []
    for _ in range(6):
        e.init_fixed(start)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        torch.cuda.synchronize()
        a.record()
        e.step(events)
        b.record()
        torch.cuda.synchronize()
        ms.append(a.elapsed_time(b))
    return min(ms)


@pytest.mark.parametrize("n_tot,k0", [(24, 0.1), (32, 0.01), (48, 0.01), (61, 0.05)])
def test_active_ensembles_keep_the_words_where_they_win(torch, n_tot, k0):
    """24576 words of few planes, every replica in its active phase (the lanes
    loop takes 1.2 to 1.4 times as long)."""
    net = bwg.Network(frank_network(n_tot, k0=k0))
    M, start = 32 * 24576, (0, 0, n_tot)
    got, words = (active_ms(torch, net, M, start, 200, **kw) for kw in ({}, dict(word_bits=32)))
    print("ms", n_tot, k0, got, words, flush=True)
    assert got < 1.15 * words


@pytest.mark.parametrize("word_bits", [0, 32], ids=["lanes", "words"])
def test_batch_queues(torch, word_bits):
    """The two persistent kernels: a batch on the lanes loop (64-word items
    taken by pairs of words, and two-word items asked for), and one that a
    given word width keeps on the word functions beside lanes items."""
    mix = [(frank_network(16, k0=0.05), 33, 12.0), (frank_network(100, k0=0.01), 4200, 3.0),
           (frank_network(40, k0=0.1), 2048, 6.0), (frank_network(1000, k0=0.02), 97, 0.75),
           (exact_network(90, 7, 0, 0), 65, 0.05)]
    ens, alone = [], []
    for k, (net, M, _) in enumerate(mix):
        for out, kw in ((ens, dict(word_bits=word_bits)), (alone, dict(engine="lanes"))):
            e = bwg.Ensemble(bwg.Network(net), M, seed=3, net_id=k, **kw)
            out.append(e.init_fixed((0, 0, net["n_tot"])))
    ens[0].set_engine("lanes")
    ens[1].set_lanes_words(70)
    b = bwg.Batch(ens, waves=100)
    t = [m[2] for m in mix]
    b.advance(t)
    for e, x in zip(ens, t):
        e.schedule(2 * x)
    while any(e.pending() for e in ens):
        b.run(250)
    for e, f, x in zip(ens, alone, t):
        f.advance(x).advance(2 * x)
        np.testing.assert_array_equal(e.read_counts().cpu().numpy(), f.read_counts().cpu().numpy())
        for u, v in zip(e.read_events(), f.read_events()):
            np.testing.assert_array_equal(u.cpu().numpy(), v.cpu().numpy())


# ---- networks on the general path ------------------------------------------------

def table(species, reactions, rates, n_tot, open_net=False):
    net = _net(reactions, rates, n_tot, exact_integer=True)
    net["species"] = tuple("S%d" % x for x in range(species))
    net["hop_rates"] = [0.0] * species
    net["open"] = open_net
    return net


GENERAL = {
    "random12": (random_network(2, 200, 12), ("multinomial",)),
    "random16": (random_network(3, 12, 16), ("multinomial",)),
    # weights and products beyond 24 bits
    "heavy": (table(3, [((2, 0, 0), (0, 1, 1)), ((0, 1, 1), (2, 0, 0)), ((0, 0, 1), (0, 1, 0))],
                    [1 << 25, 3 << 23, (1 << 26) + 5], 8), ("fixed", (3, 3, 2))),
    "crowd": (table(3, [((1, 1, 0), (0, 1, 1)), ((0, 2, 0), (1, 1, 0)), ((0, 0, 1), (1, 0, 0))],
                    [3, 2, 70000], 9000), ("fixed", (3000, 2500, 3500))),
    # a ghost between reactions that change the state, and one after them
    "ghosts": (table(3, [((1, 1, 0), (0, 1, 1)), ((1, 1, 0), (1, 1, 0)), ((0, 0, 2), (1, 1, 0)),
                         ((0, 2, 0), (0, 2, 0))], [3, 5, 2, 7], 60), ("fixed", (20, 30, 10))),
    # one to eight species, closed and open
    "one": (open_network("birth", 70), ("fixed", (3,))),
    "death": (open_network("death", 500), ("fixed", (400,))),
    "predators": (open_network("lotka_volterra", 90), ("fixed", (40, 30))),
    "wide2": (random_wide_network(4, 2, 100, 5), ("fixed", (50, 50))),
    "wide5": (random_wide_network(3, 5, 300, 10), ("fixed", (60,) * 5)),
    "wide8": (random_wide_network(9, 8, 64, 14), ("fixed", (8,) * 8)),
    # caps that block firings most of the time
    "capped4": (random_wide_network(6, 4, 9, 10, open_net=True), ("fixed", (9, 8, 9, 7))),
    "capped7": (random_wide_network(12, 7, 30, 16, open_net=True), ("fixed", (29,) * 7)),
    # a cap of one: gains of two that no state has room for, beside one that fits
    "cap1": (table(2, [((1, 0), (1, 2)), ((1, 0), (1, 1)), ((0, 1), (0, 0))], [3, 1, 2], 1,
                   open_net=True), ("fixed", (1, 0))),
    "cap1alone": (table(1, [((1,), (3,))], [1], 1, open_net=True), ("fixed", (1,))),
}


@pytest.mark.parametrize("word_bits", [0, 32], ids=["lanes", "words"])
@pytest.mark.parametrize("name", sorted(GENERAL))
def test_general_networks_on_both_kernels(torch, name, word_bits):
    net, init = GENERAL[name]
    M = 1000 + 7
    print("case", name, word_bits, bwg.Network(net).quantized()["B"], flush=True)
    e = bwg.Ensemble(bwg.Network(net), M, seed=4, net_id=9, word_bits=word_bits)
    o = ssa.OracleEnsemble(net, M, seed=4, net_id=9)
    t = 70.0 / bwg.Network(net).quantized()["Lambda"]
    for x in (e, o):
        x.init(init)
        x.step(33)
        x.advance(t)
        x.advance(4 * t)
    np.testing.assert_array_equal(e.read_counts().cpu().numpy(), o.counts)
    ev, real = e.read_events()
    np.testing.assert_array_equal(ev.cpu().numpy().astype(np.uint64), o.E)
    want = np.zeros((M + 31) // 32, np.uint64)
    np.add.at(want, np.arange(M) // 32, o.real.astype(np.uint64))
    np.testing.assert_array_equal(real.cpu().numpy().astype(np.uint64), want)


def test_real_events_of_one_launch_past_32_bits(torch):
    """L and D turn into each other, two molecules, total weight 2 = 2^B: every
    event of every replica is real, 2^32 and some of the one word in a launch."""
    net = table(3, [((1, 0, 0), (0, 1, 0)), ((0, 1, 0), (1, 0, 0))], [1, 1], 2)
    assert bwg.Network(net).quantized()["B"] == 1
    n = (1 << 27) + 5
    e = bwg.Ensemble(bwg.Network(net), 32, seed=3)
    e.init_fixed((1, 1, 0)).step(n)
    ev, real = e.read_events()
    assert (ev == n).all() and real.tolist() == [32 * n]
    assert e.stats()["real_total"] == 32 * n
    c = e.read_counts()
    assert (c[:, 0] + c[:, 1] == 2).all() and (c >= 0).all()


@pytest.mark.parametrize("M", [64, 100000])
@pytest.mark.parametrize("call", ["step", "run", "batch"])
def test_chains_of_several_launches(torch, call, M):
    """More events than one launch of the loop runs, nearly all of them after
    the chains' ends: every event counts."""
    net = bwg.Network(frank_network(5, k0=0.3))
    n = 3 * (1 << 26) + 7
    a, b = (bwg.Ensemble(net, M, seed=3, engine="lanes", table_capacity=1 << 19)
            .init_fixed((0, 0, 5)) for _ in range(2))
    b.step(20000)
    if call == "step":
        a.step(n)
    else:
        a.schedule(n / net.quantized()["Lambda"])
        runs = bwg.Batch([a]) if call == "batch" else a
        runs.run(100)
        runs.run(2 * (1 << 26) + 5)
        runs.run()
    assert a.pending() == 0
    ev, real = a.read_events()
    if call == "step":
        assert bool((ev == n).all())
    else:
        assert n - 10 ** 6 < int(ev.min()) < int(ev.max()) < n + 10 ** 6
    np.testing.assert_array_equal(a.read_counts().cpu().numpy(), b.read_counts().cpu().numpy())
    np.testing.assert_array_equal(real.cpu().numpy(), b.read_events()[1].cpu().numpy())


@pytest.mark.parametrize("turned,weight,words", [(3, 163, 65536), (3, 31, 65536), (6, 15, 65536)])
def test_active_general_networks_keep_the_words_where_they_win(torch, turned, weight, words):
    """Conversions among three species, every event real (the lanes loop takes
    1.3 times as long)."""
    turns = [((1, 0, 0), (0, 1, 0)), ((0, 1, 0), (0, 0, 1)), ((0, 0, 1), (1, 0, 0)),
             ((1, 0, 0), (0, 0, 1)), ((0, 0, 1), (0, 1, 0)), ((0, 1, 0), (1, 0, 0))][:turned]
    net = bwg.Network(table(3, turns, [weight] * turned, 100))
    got, of_words = (active_ms(torch, net, 32 * words, (33, 33, 34), 150, **kw)
                     for kw in ({}, dict(word_bits=32)))
    print("ms", turned, weight, words, got, of_words, flush=True)
    assert got < 1.15 * of_words


# both sides of the lines by weight bits times planes
@pytest.mark.parametrize("weight,turns,words", [(1, 3, 16384), (31, 3, 32768), (117, 6, 65536),
                                                (63, 6, 98304)])
@pytest.mark.parametrize("more", [0, 1])
def test_both_sides_of_the_general_rule(torch, weight, turns, words, more):
    M = 32 * words + more
    ring = [((1, 0, 0), (0, 1, 0)), ((0, 1, 0), (0, 0, 1)), ((0, 0, 1), (1, 0, 0)),
            ((1, 0, 0), (0, 0, 1)), ((0, 0, 1), (0, 1, 0)), ((0, 1, 0), (1, 0, 0))][:turns]
    net = bwg.Network(table(3, ring, [weight] * turns, 60))
    got = []
    for kw in (dict(), dict(word_bits=32)):
        e = bwg.Ensemble(net, M, seed=2, **kw).init_fixed((20, 20, 20)).step(40)
        got.append((e.read_counts(), *e.read_events()))
    for x, y in zip(*got):
        assert bool((x == y).all())


# ---- states that nothing leaves -----------------------------------------------------

@pytest.mark.parametrize("kw", [dict(engine="lanes"), dict(word_bits=32), dict(block=256),
                                dict(block=64), dict(word_bits=16), dict(word_bits=64),
                                dict(shared_threshold=True),
                                dict(shared_threshold=True, word_bits=64)],
                         ids=lambda k: "-".join("%s" % v for v in k.values()))
@pytest.mark.parametrize("M,n_tot,steps", [(65, 8, 700), (4000, 12, 900), (8192 + 3, 32, 3000)])
def test_chains_that_end_early(torch, kw, M, n_tot, steps):
    """The paper's network ends in states that no event leaves, at some event
    of its own for every replica; loops that stop there still count every
    event, and a later step finds nothing to do."""
    net = paper_network(n_tot)
    e = bwg.Ensemble(bwg.Network(net), M, seed=11, net_id=3, **kw)
    draw = ssa.DRAW_SHARED if kw.get("shared_threshold") else ssa.DRAW_EVENT
    o = ssa.OracleEnsemble(net, M, seed=11, net_id=3, draw=draw)
    for x in (e, o):
        x.init(("multinomial",))
        x.step(steps // 7)
        x.step(steps)
    for more in (1, 500):
        np.testing.assert_array_equal(e.read_counts().cpu().numpy(), o.counts)
        ev, real = e.read_events()
        np.testing.assert_array_equal(ev.cpu().numpy().astype(np.uint64), o.E)
        want = np.zeros((M + 31) // 32, np.uint64)
        np.add.at(want, np.arange(M) // 32, o.real.astype(np.uint64))
        np.testing.assert_array_equal(real.cpu().numpy().astype(np.uint64), want)
        e.step(more)
        o.step(more)
