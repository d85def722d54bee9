"""The kernels that keep a layer's slot map in LDS (np_select_delta, np_delta
and np_delta_n up to F 32768, C 16384, k 8192) at the edges of their sizes and
of their shortcuts, against the oracle, bit for bit: ids per thread (F 16384 |
16385), slots per thread (C 8192 | 8193), actives per thread (k 2048, 4096 |
+ 1), F a multiple of 4 or not, the largest layer and the first ones past it,
tokens so far apart that the victims' ages leave the histogram, scores tied
past what one bin resolves, counts from 0 to k, and ids that are no active
set (reported; nothing out of range is written)."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2608_22643_amd import binding as B
from paper_2608_22643_amd import workload as W
from gpu_util import Bufs, compare_delta, from_dev, say

pytestmark = pytest.mark.gpu

SHAPES = [  # L, F, k, C
    (2, 16384, 2048, 8192), (2, 16385, 2049, 8193), (1, 16383, 4097, 8193),
    (1, 20002, 1999, 16384), (1, 32768, 8192, 16384), (1, 32767, 4096, 9000),
    (1, 32768, 3000, 16385), (1, 32769, 3000, 9000), (3, 65, 7, 9), (2, 31, 31, 31),
]


def cfg_of(L, F, k, C):
    return W.Config("lds", L, 64, F, 8, k / F, C / F, "f32", "f32", 4, rho_given=0.9, k_override=k,
                    c_override=C)


def check_state(bufs, st):
    P, Q, U = bufs.host_state()
    assert np.array_equal(P, st.slot_of) and np.array_equal(Q, st.neuron_of)
    assert np.array_equal(U, st.last_used)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "L%d_F%d_k%d_C%d" % s)
def test_delta_lds_sizes(shape):
    L, F, k, C = shape
    cfg = cfg_of(*shape)
    say(f"[delta lds] {shape}")
    rng = np.random.default_rng(F + k)
    bufs, two = Bufs(cfg), Bufs(cfg)
    bufs.reset()
    two.reset()
    st = orc.State(L, F, C)
    s = rng.standard_normal((L, F))
    # tokens 3000 apart: some victims are more than a histogram older than others
    for i, token in enumerate((0, 1, 2, 3, 3003, 3004, 6100, 6101, 6102)):
        s = 0.9 * s + np.sqrt(1 - 0.81) * rng.standard_normal((L, F))
        v = s.astype(np.float32)
        if i in (2, 5):
            v = np.round(v * 4) / np.float32(4)  # more equal keys than a bin resolves
        if i == 6:
            v[:] = 1.5  # one value: the ids decide
        dev = torch.from_numpy(v.reshape(-1)).cuda()
        B.np_select_delta(bufs.shape, token, dev, bufs.mask, bufs.ids, bufs.state, bufs.out, bufs.ws)
        B.np_select(two.shape, dev, two.mask, two.ids, two.ws)
        B.np_delta(two.shape, token, two.ids, two.state, two.out, two.ws)
        torch.cuda.synchronize()
        mask, ids = orc.select(v, k)
        assert np.array_equal(from_dev(bufs.ids, np.int32, (L, k)), ids), i
        assert torch.equal(bufs.mask, two.mask)
        assert np.array_equal(from_dev(bufs.mask, np.uint32, mask.shape), mask), i
        ref = orc.delta(token, ids, st, C)
        for b in (bufs, two):
            compare_delta(b.host_lists(), ref, L)
            check_state(b, st)
            assert B.np_device_error(b.ws) == 0


@pytest.mark.parametrize("shape", [(3, 11008, 1651, 5504), (2, 14337, 5500, 7168)],
                         ids=["aligned", "odd"])
def test_delta_lds_counts(shape):
    """np_delta_n with counts 0 .. k against the oracle."""
    L, F, k, C = shape
    cfg = cfg_of(*shape)
    say(f"[delta lds counts] {shape}")
    rng = np.random.default_rng(5)
    bufs = Bufs(cfg)
    bufs.reset()
    st = orc.State(L, F, C)
    for token in range(6):
        counts = rng.integers(0, k + 1, size=L).astype(np.int32)
        counts[token % L] = (0, k, 1)[token % 3]
        ids = np.zeros((L, k), np.int32)
        for l in range(L):
            ids[l, :counts[l]] = np.sort(rng.choice(F, counts[l], replace=False))
        pad = np.zeros(max(L, 4), np.int32)
        pad[:L] = counts
        B.np_delta_n(bufs.shape, token, torch.from_numpy(ids).cuda(), torch.from_numpy(pad).cuda(),
                     bufs.state, bufs.out, bufs.ws)
        torch.cuda.synchronize()
        ref = orc.delta_n(token, ids, counts, st, C)
        got = bufs.host_lists()
        for l in range(L):
            assert np.array_equal(got["counts"][l], ref["counts"][l]), (token, l)
            n = counts[l]
            assert np.array_equal(got["active_slots"][l][:n], ref["active_slots"][l][:n]), (token, l)
        check_state(bufs, st)
        assert B.np_device_error(bufs.ws) == 0


@pytest.mark.parametrize("bad", ["range", "descending", "slot_range", "unpaired"])
def test_delta_lds_bad_inputs(bad):
    """Ids that are no ascending neuron ids, slots outside the layer and
    unpaired entries set NP_DEVERR_STATE; every entry stays in range."""
    L, F, k, C = 2, 11008, 300, 900
    cfg = cfg_of(L, F, k, C)
    say(f"[delta lds bad] {bad}")
    rng = np.random.default_rng(8)
    bufs = Bufs(cfg)
    bufs.reset()

    def step(token, ids):
        B.np_delta(bufs.shape, token, torch.from_numpy(ids).cuda(), bufs.state, bufs.out, bufs.ws)
        torch.cuda.synchronize()

    def draw():
        return np.stack([np.sort(rng.choice(F, k, replace=False)) for _ in range(L)]).astype(np.int32)

    for token in range(4):
        step(token, draw())
    assert B.np_device_error(bufs.ws) == 0
    ids = draw()
    if bad == "range":
        ids[0, -1] = F + 5
        ids[1, 0] = -3
    elif bad == "descending":
        ids[0, 10], ids[0, 11] = ids[0, 11], ids[0, 10]
    elif bad == "slot_range":
        bufs.slot_of.view(L, F)[1, 77] = C + 4
        ids[1] = np.sort(np.r_[77, 100 + rng.choice(F - 100, k - 1, replace=False)])
    else:
        Q = bufs.neuron_of.view(L, C)
        Q[0, 3] = (int(Q[0, 3]) + 1) % F
    if bad == "descending":  # the same set: a defined result, whatever the order
        st_ids = np.sort(ids, axis=1)
        step(4, ids)
        hit = bufs.host_lists()["active_slots"]
        P, Q, _ = bufs.host_state()
        for l in range(L):
            assert np.array_equal(P[l][ids[l]], hit[l])
            assert np.all(P[l][st_ids[l]] >= 0)
        assert B.np_device_error(bufs.ws) == 0
        return
    step(4, ids)
    assert B.np_device_error(bufs.ws) & B.NP_DEVERR_STATE
    lists = bufs.host_lists()
    assert np.all(lists["active_slots"] < C) and np.all(lists["active_slots"] >= -1)
    P, Q, _ = bufs.host_state()
    assert np.all(Q < F) and np.all(Q >= -1)


# The same layers with F padded past 32768 run delta_kernel (delta_layer, the
# state read from memory): the added ids are never active and never resident,
# so every list and the unpadded part of the state must come out the same.
PADDED_F = 33000


class Pair:
    """One state in the LDS kernels' shape and in the padded one."""

    def __init__(self, shape, P, Q, U):
        self.shape = L, F, k, C = shape
        self.lds, self.gen = Bufs(cfg_of(L, F, k, C)), Bufs(cfg_of(L, PADDED_F, k, C))
        for b, width in ((self.lds, F), (self.gen, PADDED_F)):
            b.reset()
            b.slot_of.view(L, width)[:, :F] = torch.from_numpy(P).cuda()
            b.neuron_of.copy_(torch.from_numpy(Q).reshape(-1))
            b.last_used.view(L, width)[:, :F] = torch.from_numpy(U).cuda()

    def step(self, entry, token, ids, counts=None):
        """One delta of the ids through `entry` on both; returns the lists and
        the error word, having compared everything."""
        L, F, k, C = self.shape
        dev = torch.from_numpy(ids).cuda()
        for b, width in ((self.lds, F), (self.gen, PADDED_F)):
            if entry == "select_delta":
                s = np.full((L, width), -1.0, np.float32)
                for l in range(L):
                    s[l, ids[l]] = 1.0 + ids[l] / np.float32(width)
                B.np_select_delta(b.shape, token, torch.from_numpy(s).cuda(), b.mask, b.ids, b.state,
                                  b.out, b.ws)
            elif entry == "delta_n":
                n = np.zeros(max(L, 4), np.int32)
                n[:L] = k if counts is None else counts
                B.np_delta_n(b.shape, token, dev, torch.from_numpy(n).cuda(), b.state, b.out, b.ws)
            else:
                B.np_delta(b.shape, token, dev, b.state, b.out, b.ws)
        torch.cuda.synchronize()
        got, ref = self.lds.host_lists(), self.gen.host_lists()
        compare_delta(got, ref, L)
        for x, y in zip(self.lds.host_state(), self.gen.host_state()):
            w = x.shape[1]
            assert np.array_equal(x, y[:, :w])
            assert np.all(y[:, w:] == -1)
        err = B.np_device_error(self.lds.ws)
        assert err == B.np_device_error(self.gen.ws)
        return got, err


def seeded(rng, shape, resident, never, tokens):
    """A consistent slot map with `resident` rows a layer, `never` of them
    never used, the others last used at a token of [0, tokens)."""
    L, F, k, C = shape
    P, U = np.full((L, F), -1, np.int32), np.full((L, F), -1, np.int32)
    Q = np.full((L, C), -1, np.int32)
    for l in range(L):
        n, s = rng.permutation(F)[:resident], rng.permutation(C)[:resident]
        P[l, n], Q[l, s] = s, n
        U[l, n[never:]] = rng.integers(0, tokens, resident - never)
    return P, Q, U


@pytest.mark.parametrize("entry", ["delta", "delta_n", "select_delta"])
@pytest.mark.parametrize("tokens", [50, 4000])  # ages inside and past the histogram
@pytest.mark.parametrize("never", [0.1, 1.0])
@pytest.mark.parametrize("shape", [(2, 3000, 300, 900), (2, 11008, 1651, 5504),
                                   (1, 28672, 2867, 8601)], ids=lambda s: f"F{s[1]}")
def test_delta_lds_never_used_rows(shape, never, tokens, entry):
    """A slot map that the caller seeded, full but for a few slots, a tenth or
    all of its rows never used (last_used -1): those leave first, by id."""
    L, F, k, C = shape
    say(f"[delta lds never used] {shape} {never} {tokens} {entry}")
    rng = np.random.default_rng(C + tokens)
    P, Q, U = seeded(rng, shape, C - 7, int(never * (C - 7)), tokens)
    pair = Pair(shape, P, Q, U)
    st = orc.State(L, F, C)
    st.slot_of[:], st.neuron_of[:], st.last_used[:] = P, Q, U
    for i in range(3):
        ids = np.stack([np.sort(rng.choice(F, k, replace=False)) for _ in range(L)]).astype(np.int32)
        got, err = pair.step(entry, tokens + i, ids)
        assert err == 0
        ref = orc.delta(tokens + i, ids, st, C)
        assert np.all(ref["counts"][:, 2] > 0)  # victims
        compare_delta(got, ref, L)
        check_state(pair.lds, st)


@pytest.mark.parametrize("entry", ["delta", "delta_n", "select_delta"])
@pytest.mark.parametrize("kind", ["stale_slot", "slot_range", "lost_slot", "two_slots", "neuron_range"])
@pytest.mark.parametrize("shape", [(2, 3000, 300, 900), (2, 11008, 1651, 5504),
                                   (1, 28672, 2867, 8601)], ids=lambda s: f"F{s[1]}")
def test_delta_lds_inconsistent_state(shape, kind, entry):
    """A slot map with a twentieth of its entries wrong, in a full buffer: the
    LDS kernels' checked path gives every list, every state entry and the error
    word that the kernel of its own for larger layers gives."""
    L, F, k, C = shape
    say(f"[delta lds inconsistent] {shape} {kind} {entry}")
    rng = np.random.default_rng(C)
    P, Q, U = seeded(rng, shape, C - 7, 5, 50)
    for l in range(L):
        held = rng.choice(np.flatnonzero(P[l] >= 0), C // 20, replace=False)
        free = rng.choice(np.flatnonzero(P[l] < 0), C // 20, replace=False)
        if kind == "stale_slot":  # a neuron names a slot that another holds
            P[l, free] = P[l, held]
        elif kind == "slot_range":
            P[l, free] = C + 4 + np.arange(len(free))
            P[l, held[::2]] = -3
        elif kind == "lost_slot":  # a slot names a neuron that does not know
            P[l, held] = -1
        elif kind == "two_slots":  # two slots name the same neuron
            Q[l, P[l, held[::2]]] = held[1::2][:len(held[::2])][0]
        else:
            Q[l, P[l, held[::2]]] = F + 3
            Q[l, P[l, held[1::2]]] = -5
    pair = Pair(shape, P, Q, U)
    for i in range(3):
        ids = np.stack([np.sort(rng.choice(F, k, replace=False)) for _ in range(L)]).astype(np.int32)
        got, err = pair.step(entry, 50 + i, ids)
        assert np.all(got["counts"][:, 2] > 0)
        if i == 0:
            assert err == B.NP_DEVERR_STATE


@pytest.mark.parametrize("shape", [(2, 3000, 300, 900), (2, 11008, 1651, 5504)], ids=lambda s: f"F{s[1]}")
def test_delta_lds_bad_counts_and_order(shape):
    """Counts outside [0, k] and ids in descending order, against the kernel
    for larger layers."""
    L, F, k, C = shape
    say(f"[delta lds counts and order] {shape}")
    rng = np.random.default_rng(C)
    pair = Pair(shape, *seeded(rng, shape, C - 7, 5, 50))
    for i, counts in enumerate((None, [k + 3, k], [-2, k // 2])):
        ids = np.stack([np.sort(rng.choice(F, k, replace=False)) for _ in range(L)]).astype(np.int32)
        _, err = pair.step("delta_n", 50 + i, ids, counts)
        assert (err != 0) == (i > 0)
    ids = np.stack([np.sort(rng.choice(F, k, replace=False))[::-1] for _ in range(L)]).astype(np.int32)
    pair.step("delta", 60, np.ascontiguousarray(ids))
