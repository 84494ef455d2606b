"""The transform-domain blind rotation (the automatic schedule at N = 1024)
against the stream-ordered int8 kernels and the oracle, word for word (needs
an MI355X).  Short LWE dimensions keep the key small; the ring is the Table 7
one, the only one this schedule runs."""
import struct

import numpy as np
import pytest

from oracle import params as OP
from oracle import tfhe
from tests import helpers

pytestmark = pytest.mark.gpu

AUTO, STREAM, PERSISTENT = -1, 0, 1


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def _params(k, n, ell):
    return OP.Params(k=k, n=n, N=1024, bk_ell=ell, ks_t=8, bk_noise_log2=30, ks_noise_log2=15, lwe_noise_log2=15)


def _world(P, seed):
    import paper_2205_05825_amd as mk
    ctx = mk.Context(helpers.lib_params(P), seed)
    for i in range(P.k):
        ctx.keygen(i, tfhe.party_seed(seed, i))
    return ctx


def _rotate(torch, ctx, abar, steps, kind):
    P = ctx.params
    ta = torch.from_numpy(np.ascontiguousarray(abar).view(np.int32)).to("cuda:0")
    acc = torch.full((len(abar), (P.k + 1) * P.N), 5, dtype=torch.int32, device="cuda:0")
    ctx.set_rotation(kind)
    try:
        ctx.blind_rotate(ta, acc, max_steps=steps)
    finally:
        ctx.set_rotation(AUTO)
    torch.cuda.synchronize()
    return acc.cpu().numpy().view(np.uint32)


def _abar(P, cnt, seed):
    a = np.random.default_rng(seed).integers(0, 2 * P.N, (cnt, P.lwe_words)).astype(np.uint32)
    a[0, :] = 0                      # every step adds zero
    a[-1, :] = 2 * P.N - 1
    a[cnt // 2, 1::2] = 0
    a[cnt // 3, :] = P.N
    return a


@pytest.mark.parametrize("k,ell", [(1, 3), (2, 3), (2, 1), (2, 2), (3, 3), (4, 3), (5, 2), (8, 3)])
def test_party_counts_and_gadget_lengths(torch_cuda, k, ell):
    """Every accumulator word equals the stream-ordered schedule's for one
    gate and for counts on both sides of the one-gate-per-compute-unit limit
    (up to 2 rounds of 256 at k <= 2), across every party boundary, and the
    oracle's on a few gates."""
    P = _params(k, 5, ell)
    ctx = _world(P, 40 + k)
    ctx.upload()
    K = tfhe.generate(P, 40 + k)
    for cnt in (1, 3, 257, 514):
        abar = _abar(P, cnt, 10 * k + cnt)
        got = _rotate(torch_cuda, ctx, abar, -1, AUTO)
        assert np.array_equal(got, _rotate(torch_cuda, ctx, abar, -1, STREAM)), cnt
        if cnt == 3:
            for g in range(cnt):
                assert np.array_equal(got[g].reshape(k + 1, P.N), tfhe.blind_rotate(K, abar[g].astype(np.int64))), g
    ctx.close()


@pytest.mark.parametrize("steps", [0, 1, 4, 7])
def test_partial_rotations(torch_cuda, steps):
    """max_steps from none to across the party boundary, both kernels."""
    P = _params(2, 6, 3)
    ctx = _world(P, 50)
    ctx.upload()
    for cnt in (2, 600):
        abar = _abar(P, cnt, steps + cnt)
        assert np.array_equal(_rotate(torch_cuda, ctx, abar, steps, AUTO),
                              _rotate(torch_cuda, ctx, abar, steps, STREAM)), cnt
    ctx.close()


@pytest.mark.parametrize("k,pattern", [(2, "min"), (2, "max"), (2, "halves"), (2, "alternate"), (8, "halves")])
def test_extreme_keys(torch_cuda, k, pattern):
    """Imported key polynomials at the ends of both 16-bit halves, constant
    (every product concentrated on one result and frequency) or alternating:
    the largest sums the rounding has to get right.  Every word equals the
    exact int8 schedule's."""
    P = _params(k, 4, 3)
    ctx = _world(P, 60)
    words = {"min": [0x80000000], "max": [0x7FFF7FFF], "halves": [0x80008000],
             "alternate": [0x7FFF7FFF, 0x80008000]}[pattern]
    head = 4 + 4 + 40 + 4
    for party in range(k):
        data = bytearray(ctx.export_keys(party))
        assert struct.unpack_from("<4s", data)[0] == b"MKK1"
        pk = head + P.n + P.N
        polys = 3 + P.n * 9
        fill = np.tile(np.array(words, np.uint32), polys * P.N // len(words))
        data[pk:pk + 4 * polys * P.N] = fill.tobytes()
        ctx.import_keys(party, bytes(data))
    ctx.upload()
    for cnt in (2, 520):
        abar = _abar(P, cnt, cnt)
        assert np.array_equal(_rotate(torch_cuda, ctx, abar, -1, AUTO), _rotate(torch_cuda, ctx, abar, -1, STREAM)), cnt
    ctx.close()


@pytest.mark.parametrize("k,n,cnt", [(2, 70, 3), (2, 5, 72), (2, 5, 73), (3, 5, 80), (4, 5, 81), (8, 4, 7),
                                     (8, 4, 64), (8, 4, 73)])
def test_teams_of_workgroups(torch_cuda, k, n, cnt):
    """Batches narrow enough for several workgroups per gate, at the limits of
    each team size (slots shared out to helpers and left with members 0 and
    1) and past 64 steps of a party, twice over on one context: every word
    equals the stream-ordered schedule's."""
    P = _params(k, n, 3)
    ctx = _world(P, 70 + k)
    ctx.upload()
    for seed in (1, 2):
        abar = _abar(P, cnt, seed)
        assert np.array_equal(_rotate(torch_cuda, ctx, abar, -1, AUTO), _rotate(torch_cuda, ctx, abar, -1, STREAM)), seed
    ctx.close()


@pytest.mark.parametrize("k,cnt", [(2, 300), (2, 1090), (4, 800), (8, 280)])
def test_batches_in_parts(torch_cuda, k, cnt):
    """Batches whose last gates run on another kernel than the full rounds
    before them: every word equals the stream-ordered schedule's."""
    P = _params(k, 3, 3)
    ctx = _world(P, 80 + k)
    ctx.upload()
    abar = _abar(P, cnt, cnt)
    assert np.array_equal(_rotate(torch_cuda, ctx, abar, -1, AUTO), _rotate(torch_cuda, ctx, abar, -1, STREAM))
    ctx.close()


@pytest.mark.parametrize("k,cnt", [(2, 3), (2, 300), (2, 600)])
def test_amounts_inside_the_accumulators(torch_cuda, k, cnt):
    """Rotation amounts that lie in the buffer the accumulators are written to:
    every word equals the rotation's with the amounts elsewhere."""
    P = _params(k, 5, 3)
    ctx = _world(P, 90 + k)
    ctx.upload()
    abar = _abar(P, cnt, cnt)
    want = _rotate(torch_cuda, ctx, abar, -1, AUTO)
    for at in (0, cnt * (P.k + 1) * P.N - abar.size):   # first and last words of the buffer
        buf = torch_cuda.full((cnt, (P.k + 1) * P.N), 5, dtype=torch_cuda.int32, device="cuda:0")
        inside = buf.view(-1)[at:at + abar.size].view(abar.shape)
        inside.copy_(torch_cuda.from_numpy(abar.view(np.int32)))
        ctx.blind_rotate(inside, buf)
        torch_cuda.cuda.synchronize()
        assert np.array_equal(buf.cpu().numpy().view(np.uint32), want), at
    ctx.close()


@pytest.mark.parametrize("k,n,cnt", [(2, 5, 1), (2, 70, 73), (4, 5, 40), (8, 4, 64)])
def test_teams_given_up(torch_cuda, k, n, cnt):
    """A team whose members do not all run in time is left to one workgroup per
    gate.  Waits of no, a few and the usual number of polls in turn on one
    context: every word equals the stream-ordered schedule's, and no rotation
    reports a time-out."""
    P = _params(k, n, 3)
    ctx = _world(P, 100 + k)
    ctx.upload()
    abar = _abar(P, cnt, cnt)
    want = _rotate(torch_cuda, ctx, abar, -1, STREAM)
    for polls in (0, 1, 3, -1, 0):
        ctx.set_team_wait(polls)
        assert np.array_equal(_rotate(torch_cuda, ctx, abar, -1, AUTO), want), polls
        ctx.device_status()
    ctx.close()


@pytest.mark.parametrize("kind,rows", [(AUTO, 0), (PERSISTENT, 2)])
def test_teams_beside_another_context(torch_cuda, kind, rows):
    """Narrow batches on one context and stream while another context keeps
    every compute unit busy on its own (several gates per compute unit, or
    persistent teams of 32): both give the words they give alone."""
    torch = torch_cuda
    P = _params(2, 40, 3)
    narrow, wide = _world(P, 110), _world(P, 111)
    narrow.upload()
    wide.upload()
    wide.set_rotation(kind)
    wide.set_team_rows(rows)
    a = [torch.from_numpy(_abar(P, cnt, cnt).view(np.int32)).to("cuda:0") for cnt in (1, 64, 1500)]
    accs = [torch.zeros((len(x), (P.k + 1) * P.N), dtype=torch.int32, device="cuda:0") for x in a]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    want = []
    for i, x in enumerate(a):
        (wide if i == 2 else narrow).blind_rotate(x, accs[i])
        torch.cuda.synchronize()
        want.append(accs[i].clone())
        accs[i].zero_()
    torch.cuda.synchronize()
    for _ in range(4):
        wide.blind_rotate(a[2], accs[2], stream=streams[1])
        for i in (0, 1):
            narrow.blind_rotate(a[i], accs[i], stream=streams[0])
    torch.cuda.synchronize()
    for i in range(3):
        assert torch.equal(accs[i], want[i]), i
    narrow.device_status()
    wide.device_status()
    narrow.close()
    wide.close()


@pytest.mark.parametrize("n,batch", [(560, 3), (511, 140)])
def test_largest_graph_pieces(torch_cuda, n, batch):
    """Circuits captured in pieces of up to the largest size, at a rotation
    longer than a piece (1120 steps count as 4480 kernels) and one that nearly
    fills it (1022: 4088, to which the level's other kernels are added), on
    teams and on one workgroup per gate: two replays equal the eager words."""
    import paper_2205_05825_amd as mk
    P = _params(2, n, 3)
    ctx = _world(P, 120)
    ctx.upload()
    circ = mk.build_operator(mk.OP_ADD, 2)
    rng = np.random.default_rng(n)
    rows = np.stack([ctx.encrypt(i % 2, rng.integers(0, 2, batch).astype(np.uint8), seed=500 + i)
                     for i in range(len(circ.inputs))])
    inp = torch_cuda.from_numpy(rows.view(np.int32)).to("cuda:0")
    want = torch_cuda.zeros((len(circ.outputs), batch, inp.shape[2]), dtype=torch_cuda.int32, device="cuda:0")
    ctx.eval_circuit(circ, inp, want)
    for piece in (4093, 4094, 4096):
        out = torch_cuda.zeros_like(want)
        ctx.set_graph_piece(piece)
        g = ctx.circuit_graph(circ, inp, out)
        assert g.info()[2] >= mk.circuit_stats(circ)[0] * 8 * n // 4096
        for _ in range(2):
            out.zero_()
            g.launch()
            torch_cuda.cuda.synchronize()
            assert torch_cuda.equal(out, want), piece
        g.close()
    ctx.close()


@pytest.mark.parametrize("k,cnt", [(1, 32), (1, 64), (2, 25), (2, 32), (2, 64), (3, 64)])
def test_team_scratch(torch_cuda, k, cnt):
    """Counts whose boxes need more than the int8 kernels' scratch of that
    many gates: eagerly (twice, on scratch that grows), in the fixed block and
    captured, every word equals the stream-ordered schedule's."""
    import paper_2205_05825_amd as mk
    P = _params(k, 5, 3)
    ctx = _world(P, 130 + k)
    ctx.upload()
    d = "cuda:0"
    rng = np.random.default_rng(cnt)
    a, b = (torch_cuda.from_numpy(rng.integers(0, 1 << 32, (cnt, P.lwe_words), dtype=np.uint64).astype(np.uint32)
                                  .view(np.int32)).to(d) for _ in range(2))
    types = torch_cuda.full((cnt,), mk.XOR, dtype=torch_cuda.uint8, device=d)

    def gates(noalloc=False):
        out = torch_cuda.zeros_like(a)
        ctx.bootstrap_gate(types, a, b, out, noalloc=noalloc)
        return out

    got = [gates(), gates(), gates(noalloc=True)]
    io = torch_cuda.stack([a, b])
    out = torch_cuda.zeros((1,) + tuple(a.shape), dtype=torch_cuda.int32, device=d)
    g = ctx.circuit_graph(mk.Circuit(5, [2, 3], [4], np.array([[mk.XOR, 2, 3, 4]])), io, out)
    for _ in range(2):
        out.zero_()
        g.launch()
        torch_cuda.cuda.synchronize()
        got.append(out[0].clone())
    g.close()
    ctx.set_rotation(STREAM)
    want = gates()
    torch_cuda.cuda.synchronize()
    for i, x in enumerate(got):
        assert torch_cuda.equal(x, want), i
    ctx.close()


def test_upload_without_room_for_the_transforms(torch_cuda):
    """A device whose free memory holds the int8 kernels' keys but not the
    transformed ones (660 MB here; half of that is left): the upload succeeds,
    the automatic schedule runs the int8 kernels, with the same words."""
    torch = torch_cuda
    P = _params(8, 560, 3)
    transformed = P.k * P.n * 3 * P.bk_ell * 16384
    abar = _abar(P, 2, 1)
    ctx = _world(P, 140)
    free = torch.cuda.mem_get_info()[0]
    ctx.upload()
    need = free - torch.cuda.mem_get_info()[0]
    assert ctx.get_team_rows(256) == 0
    want = _rotate(torch, ctx, abar, 600, AUTO)
    ctx.close()
    ctx = _world(P, 140)
    torch.cuda.empty_cache()
    room = torch.empty(need - transformed // 2, dtype=torch.uint8, device="cuda:0")
    taken = []
    for size in (8 << 30, 512 << 20, 64 << 20):     # whatever else is free
        try:
            while True:
                taken.append(torch.empty(size, dtype=torch.uint8, device="cuda:0"))
        except torch.cuda.OutOfMemoryError:
            pass
    del room
    torch.cuda.empty_cache()
    ctx.upload()
    del taken
    torch.cuda.empty_cache()
    assert ctx.get_team_rows(256) > 0
    assert np.array_equal(_rotate(torch, ctx, abar, 600, AUTO), want)
    ctx.close()


@pytest.mark.parametrize("k,cnt", [(2, 1025), (3, 769), (3, 1024), (4, 1024), (8, 257)])
def test_what_full_rounds_leave_over(torch_cuda, k, cnt):
    """Batches just over and far over full rounds of several gates per compute
    unit: whole on that kernel at 2 parties, the rest on one gate per compute
    unit or on teams from 3 on.  Every word equals the stream-ordered
    schedule's."""
    P = _params(k, 3, 3)
    ctx = _world(P, 150 + k)
    ctx.upload()
    abar = _abar(P, cnt, cnt)
    assert np.array_equal(_rotate(torch_cuda, ctx, abar, -1, AUTO), _rotate(torch_cuda, ctx, abar, -1, STREAM))
    ctx.close()
