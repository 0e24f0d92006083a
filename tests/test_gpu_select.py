"""Global top-W beam selection (Sec. 2.1) on the GPU against the oracle.

Indices and scores are compared bit for bit: the order is total (score desc,
flat index asc, -0.0 below +0.0, NaN last), so the result is unique, and the
candidate score is one fp32 addition on both sides."""
import zlib

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2609_12399_amd import onela as ab
from paper_2609_12399_amd.workload import SELECT_CODEBOOK, make_select_inputs

pytestmark = pytest.mark.gpu

# (name, R, W_prev, V, W, kind, with_beam).  A name that begins with a form of the
# selection (one_pass, stream, two_pass; stream_N_rounds, two_pass_summary_rowsN)
# is held to it: the form that the call took is read from the workspace.  The forms
# are chosen for the 256 compute units of the whole device.
CASES = [
    ("tiny_direct", 1, 3, 5, 7, "ties", False),
    ("one_chunk_max_width", 2, 8, 2048, 4096, "logsoftmax", True),
    ("headline_w512", 1, 512, SELECT_CODEBOOK, 512, "logsoftmax", True),
    ("ragged_ties", 3, 37, 1001, 300, "ties", True),
    ("special_values", 2, 64, 300, 4096, "special", False),
    ("special_values_beam", 1, 300, 333, 1000, "special", True),
    ("keep_all", 1, 8, 125, 1000, "ties", True),
    ("one_pass_width_one", 2, 100, 999, 1, "logsoftmax", True),
    ("many_stages_w4096", 1, 1024, 4096, 4096, "ties", True),
    ("r4_w1024", 4, 1024, 4096, 1024, "logsoftmax", True),
    ("chunk_plus_one", 1, 1, 16385, 17, "ties", False),
    # one launch with a cross-workgroup bound (all chunks resident at once):
    # heavy ties, ragged last chunk, ties cut off after the chunk where W tied
    # candidates are guaranteed, special values over two requests, rising scores up
    # to the widest result it takes
    ("one_pass_ties_w512", 1, 512, SELECT_CODEBOOK, 512, "ties", True),
    ("one_pass_ties_slot_overflow", 1, 512, SELECT_CODEBOOK, 64, "ties", True),
    ("one_pass_rising_w512", 1, 512, SELECT_CODEBOOK, 512, "rising", True),
    ("one_pass_ragged", 1, 500, 8000, 300, "logsoftmax", True),
    ("one_pass_ties_w64", 1, 300, SELECT_CODEBOOK, 64, "ties", True),
    ("one_pass_r2_special", 2, 100, SELECT_CODEBOOK, 200, "special", True),
    ("one_pass_rising_w1024", 1, 1024, 4096, 1024, "rising", True),
    # many requests in one launch: a polling workgroup and a bound word per
    # request, one epoch (64 requests: every word of the control block)
    ("one_pass_r32_ties", 32, 8, SELECT_CODEBOOK, 16, "ties", True),
    ("one_pass_r64", 64, 4, SELECT_CODEBOOK, 8, "logsoftmax", True),
    # streaming form (more chunks than fit at once): rows that straddle a wave's
    # piece and a ragged last chunk with special values, rows shorter than a
    # workgroup, no beam scores, a row per 16 lanes' and per wave's summaries, slots
    # that overflow, W = 1, one workgroup with fewer chunks than the others; then a
    # last range of one candidate and of one more than a chunk, 57 short rows in a
    # range, and 4, 7 and 13 rounds (13: odd rows with special values)
    ("stream_2_rounds_special_r2", 2, 600, 4096, 256, "special", True),
    ("stream_2_rounds_ragged", 3, 1023, 2047, 500, "logsoftmax", True),
    ("stream_2_rounds_width_one_no_beam", 2, 700, 3000, 1, "logsoftmax", False),
    ("stream_4_rounds_r8_ties", 8, 256, SELECT_CODEBOOK, 256, "ties", True),
    ("stream_4_rounds_rising_r8", 8, 256, SELECT_CODEBOOK, 256, "rising", True),
    ("stream_4_rounds_r2", 2, 1024, SELECT_CODEBOOK, 256, "logsoftmax", True),
    ("stream_special_ragged", 3, 500, 3001, 200, "special", True),
    ("stream_short_rows", 3, 5000, 300, 128, "logsoftmax", True),
    ("stream_no_beam", 5, 108, SELECT_CODEBOOK, 150, "special", False),
    ("stream_wave_summaries", 1, 530, SELECT_CODEBOOK, 200, "logsoftmax", True),
    ("stream_rising_overflow", 4, 133, SELECT_CODEBOOK, 40, "rising", True),
    ("stream_ties_overflow", 4, 131, SELECT_CODEBOOK, 33, "ties", True),
    ("stream_width_one", 9, 60, SELECT_CODEBOOK, 1, "logsoftmax", True),
    ("stream_last_one", 4, 1, 68 * 16384 + 1, 20, "special", True),
    ("stream_last_chunk_and_one", 4, 1, 69 * 16384 + 1, 20, "ties", True),
    ("stream_rows_of_576", 4, 2000, 576, 60, "logsoftmax", True),
    ("stream_4_rounds", 8, 250, SELECT_CODEBOOK, 256, "logsoftmax", True),
    ("stream_4_rounds_ties", 4, 64, 65536, 64, "ties", True),
    ("stream_7_rounds_rising", 60, 50, 8000, 16, "rising", True),
    ("stream_13_rounds_special", 50, 101, 9973, 11, "special", True),
    # two passes (more survivors expected than the streaming form is for, more than
    # 64 requests, more than 512 chunks): wave maxima, then (from four rounds of
    # workgroups on) summaries with 2, 4 and 8 rows per thread; special values,
    # ragged, rising, without beam scores, ranked by the placing kernel and, beyond
    # 512 chunks, by the ranking one
    ("two_pass_rising_r2_w1024", 2, 1024, 4096, 1024, "rising", True),
    ("two_pass_placed_r80", 80, 4, SELECT_CODEBOOK, 8, "ties", True),
    ("two_pass_special_w1024", 2, 1024, 4096, 1024, "special", True),
    ("two_pass_ragged_no_beam", 2, 1023, 4099, 1000, "special", False),
    ("two_pass_r70_width_one", 70, 9, SELECT_CODEBOOK, 1, "special", True),
    ("two_pass_550_chunks", 1, 1100, SELECT_CODEBOOK, 300, "special", True),
    ("two_pass_summary_rows2_special", 17, 128, SELECT_CODEBOOK, 256, "special", True),
    ("two_pass_summary_rows2_ties_no_beam", 17, 129, 8179, 256, "ties", False),
    ("two_pass_summary_rows4_ties", 4, 1024, 4096, 1024, "ties", True),
    ("two_pass_summary_rows4_special_no_beam", 4, 1024, 4096, 1000, "special", False),
    ("two_pass_summary_rows8_special", 2, 1024, SELECT_CODEBOOK, 400, "special", True),
    ("two_pass_summary_rows8_rising_no_beam", 2, 1024, 8191, 500, "rising", False),
]


def _layout(sel):
    """(chunks per request, and the workspace offsets of the two-pass summaries
    or maxima, the bound words and the survivor counts) of a call that is large
    enough for the one-pass, streaming and two-pass forms."""
    nchunks = -(-sel.prev_width * sel.vocab // 16384)
    cap = max(64, 1 << (2 * sel.width - 1).bit_length())
    if cap > 4096:
        cap = max(4096, 1 << (sel.width - 1).bit_length())
    up = lambda x: -(-x // 256) * 256
    seg = 1024 + 8192 * 16
    bound = seg + up(sel.R * nchunks * 8 * 16)
    counts = bound + up(sel.R * 8) + up(sel.R * nchunks * cap * 8)
    return nchunks, seg, bound, counts


def _words(sel, off, n):
    return sel.workspace[off:off + 4 * n].cpu().numpy().view(np.uint32)


def _counts(sel):
    """The survivors that each chunk's slot holds after a call of one of the
    three forms, [R][nchunks], and the words beside them (largest keys)."""
    nchunks, _, _, off = _layout(sel)
    w = _words(sel, off, sel.R * nchunks * 2).reshape(sel.R, nchunks, 2)
    return w[:, :, 0], w[:, :, 1]


def _path(sel):
    """The form that the first call on a zero-filled workspace took, from what it
    left there: a call counter of 1 and tagged summaries (one-pass, which
    also stores its chunks' largest keys, and streaming), bound words (two-pass with
    summaries, with the rows of them per thread), wave maxima (two-pass), or none
    of these (reduction tree).  Of the streaming form also the rounds per
    workgroup."""
    n = sel.prev_width * sel.vocab
    if n <= 16384 or n < 4096 * sel.width:
        return "tree"
    nchunks, seg, bound, _ = _layout(sel)
    if _words(sel, 0, 1)[0] == 1:
        if _counts(sel)[1].any():
            return "one_pass"
        tagged = 0
        for M, m, km, tag in _words(sel, 1024, 8192 * 4).reshape(-1, 4).tolist():
            tagged += (tag ^ _mix(M, m, km)) == 1
        for spc in (32, 8):  # summaries per workgroup
            groups, rest = divmod(tagged, sel.R * spc)
            if rest == 0 and groups <= nchunks:
                per = -(-nchunks // groups)
                if -(-nchunks // per) == groups:
                    return f"stream_{per}_rounds"
        return "stream"
    if _words(sel, bound, 2 * sel.R).any():
        rows = 2 if nchunks <= 128 else 4 if nchunks <= 256 else 8
        return f"two_pass_summary_rows{rows}"
    return "two_pass" if _words(sel, seg, sel.R * nchunks * 8).any() else "tree"


def _run(R, P, V, W, kind, with_beam, seed):
    import torch
    from paper_2609_12399_amd.runner import BeamSelector
    logp, beam = make_select_inputs(R, P, V, seed, kind, with_beam)
    print(f"select R={R} W_prev={P} V={V} W={W} kind={kind} beam={with_beam}", flush=True)
    sel = BeamSelector(R, P, V, W)
    dl = torch.from_numpy(logp).cuda()
    db = None if beam is None else torch.from_numpy(beam).cuda()
    par, tok, sc = sel(dl, db)
    torch.cuda.synchronize()
    path = _path(sel)
    print(f"  path {path}", flush=True)
    return logp, beam, par.cpu().numpy(), tok.cpu().numpy(), sc.cpu().numpy(), path


@pytest.mark.parametrize("name,R,P,V,W,kind,with_beam", CASES, ids=[c[0] for c in CASES])
def test_select_matches_oracle(name, R, P, V, W, kind, with_beam):
    logp, beam, par, tok, sc, path = _run(R, P, V, W, kind, with_beam,
                                          seed=zlib.crc32(name.encode()) % 1000)
    for form in ("one_pass", "stream", "two_pass"):
        if name.startswith(form):
            assert path.startswith(form), path
            if "_rounds" in name or "_rows" in name and form == "two_pass":
                assert name.startswith(path), path
            elif form == "two_pass":
                assert path == "two_pass", path
    for r in range(R):
        op, ot, osc = orc.select_beams(logp[r], W, None if beam is None else beam[r])
        assert np.array_equal(par[r], op), f"request {r}: parents differ"
        assert np.array_equal(tok[r], ot), f"request {r}: tokens differ"
        assert np.array_equal(sc[r].view(np.int32), osc.view(np.int32)), \
            f"request {r}: scores differ"


@pytest.mark.parametrize("tied_slots,better", [(2, 0), (3, 0), (6, 0), (6, 300), (12, 0), (14, 200),
                                               (32, 0)])
def test_select_one_pass_many_tied_survivors(tied_slots, better):
    """Ties held by the first lane of every wave (a chunk's candidate at slot
    i of lane t sits at position 512 i + t): each wave then guarantees one
    candidate at the tied key, so all chunks up to c* (the 64th) keep every
    tied candidate of theirs, 64 x 8 x tied_slots survivors: 1024 are
    ranked by direct comparison, more too as far as they are staged, with
    `better` distinct scores above them or none (the histogram's largest bin
    holds the ties); 16384 are more than the final stage stages at all (the
    exact top-W cut over the slots).  The result is the `better` scores and the
    tied candidates with the lowest flat indices."""
    import torch
    from paper_2609_12399_amd.runner import BeamSelector
    R, P, V, W = 1, 512, SELECT_CODEBOOK, 512
    rng = np.random.default_rng(7 + tied_slots)
    logp = (-1.0 - rng.random(P * V, dtype=np.float32)).astype(np.float32)
    q = np.arange(P * V)
    logp[(q % 64 == 0) & ((q % 16384) // 512 < tied_slots)] = 0.0
    up = rng.permutation(P * V)[:better]
    logp[up] = 1.0 + rng.random(better, dtype=np.float32)
    logp = logp.reshape(R, P, V)
    print(f"one-pass tied survivors: {64 * 8 * tied_slots}, {better} above", flush=True)
    sel = BeamSelector(R, P, V, W)
    par, tok, sc = sel(torch.from_numpy(logp).cuda(), None)
    torch.cuda.synchronize()
    op, ot, osc = orc.select_beams(logp[0], W, None)
    assert np.array_equal(par.cpu().numpy()[0], op)
    assert np.array_equal(tok.cpu().numpy()[0], ot)
    assert np.array_equal(sc.cpu().numpy()[0].view(np.int32), osc.view(np.int32))


@pytest.mark.parametrize("at", ["minus_zero", "plus_zero"])
@pytest.mark.parametrize("R,P,V,W", [(1, 300, SELECT_CODEBOOK, 64), (3, 500, 3001, 200),
                                     (2, 1024, 4096, 1024), (2, 37, 1001, 300)],
                         ids=["one_pass", "stream", "two_pass", "tree"])
def test_select_signed_zeros_at_the_bound(R, P, V, W, at):
    """-0.0 orders below +0.0, and a comparison of floats does not see it.
    Nearly all scores are -0.0, with fewer than W numbers above them in every
    chunk of 16384, so that the chunks' slots overflow with zeros: either the
    bound is -0.0, or every chunk has W / 4 +0.0 and the bound is +0.0."""
    import torch
    from paper_2609_12399_amd.runner import BeamSelector
    rng = np.random.default_rng(11)
    logp = np.full((R, P * V), -0.0, dtype=np.float32)
    for r in range(R):
        for base in range(0, P * V, 16384):
            q = base + rng.permutation(min(16384, P * V - base))
            logp[r, q[:3]] = rng.random(min(3, q.size)) + 0.5
            if at == "plus_zero":
                logp[r, q[3:3 + W // 4]] = 0.0
    logp = logp.reshape(R, P, V)
    print(f"signed zeros R={R} W_prev={P} V={V} W={W} {at}", flush=True)
    par, tok, sc = BeamSelector(R, P, V, W)(torch.from_numpy(logp).cuda(), None)
    torch.cuda.synchronize()
    _check(logp, None, W, par.cpu().numpy(), tok.cpu().numpy(), sc.cpu().numpy())


@pytest.mark.parametrize("R,P,V,W", [(4, 64, 65536, 64), (16, 16, 131072, 16)])
def test_select_streaming_samples_every_part_of_the_rows(R, P, V, W):
    """The streaming form takes its bound from the first round of each
    workgroup's reads.  With the better tokens in the middle half of a
    vocabulary that is as long as a workgroup's range, whole chunks as rounds would
    sample the outer quarters only, and nearly all slots would overflow and
    be cut to W; a sample of all parts leaves a few times W survivors (expected
    about 5 W, 16 W allowed)."""
    import torch
    from paper_2609_12399_amd.runner import BeamSelector
    rng = np.random.default_rng(3)
    logp = (rng.standard_normal((R, P, V), dtype=np.float32) * 2).astype(np.float32)
    logp[:, :, V // 4:3 * V // 4] += 8.0
    beam = np.zeros((R, P), dtype=np.float32)
    print(f"sampled parts R={R} W_prev={P} V={V} W={W}", flush=True)
    sel = BeamSelector(R, P, V, W)
    par, tok, sc = sel(torch.from_numpy(logp).cuda(), torch.from_numpy(beam).cuda())
    torch.cuda.synchronize()
    _check(logp, beam, W, par.cpu().numpy(), tok.cpu().numpy(), sc.cpu().numpy())
    kept = _counts(sel)[0].sum(axis=1)
    assert (kept >= W).all() and (kept <= 16 * W).all(), kept


@pytest.mark.parametrize("W", [40, 256])
def test_select_streaming_many_ties_beyond_the_staged_ones(W):
    """More tied survivors than the placing kernel stages, in slots that are not
    in index order (a range's rounds interleave): the lowest flat indices are
    kept."""
    import torch
    from paper_2609_12399_amd.runner import BeamSelector
    R, P, V = 8, 256, SELECT_CODEBOOK
    rng = np.random.default_rng(5)
    logp = (-1.0 - rng.random((R, P * V), dtype=np.float32)).astype(np.float32)
    logp[:, rng.permutation(P * V)[:P * V // 3]] = 0.5
    logp[0, rng.permutation(P * V)[:W // 2]] = 1.0
    logp = logp.reshape(R, P, V)
    print(f"tied survivors, streaming W={W}", flush=True)
    sel = BeamSelector(R, P, V, W)
    par, tok, sc = sel(torch.from_numpy(logp).cuda(), None)
    torch.cuda.synchronize()
    _check(logp, None, W, par.cpu().numpy(), tok.cpu().numpy(), sc.cpu().numpy())


def test_select_all_equal_keeps_lowest_indices():
    import torch
    from paper_2609_12399_amd.runner import BeamSelector
    R, P, V, W = 2, 64, 1000, 777
    logp = np.full((R, P, V), -1.5, dtype=np.float32)
    sel = BeamSelector(R, P, V, W)
    par, tok, sc = sel(torch.from_numpy(logp).cuda())
    torch.cuda.synchronize()
    flat = par.cpu().numpy().astype(np.int64) * V + tok.cpu().numpy()
    assert np.array_equal(flat, np.tile(np.arange(W), (R, 1)))


def test_select_deterministic_and_feeds_resolve():
    """Repeated calls give identical bits; the parents it produces are valid
    input of the ancestry update (all in [0, W_prev))."""
    R, P, V, W = 1, 512, SELECT_CODEBOOK, 512
    a = _run(R, P, V, W, "logsoftmax", True, seed=5)
    b = _run(R, P, V, W, "logsoftmax", True, seed=5)
    for x, y in zip(a[2:5], b[2:5]):
        assert np.array_equal(x.view(np.int32), y.view(np.int32))
    assert a[2].min() >= 0 and a[2].max() < P


def _check(logp, beam, W, par, tok, sc):
    for r in range(logp.shape[0]):
        op, ot, osc = orc.select_beams(logp[r], W, None if beam is None else beam[r])
        assert np.array_equal(par[r], op), f"request {r}: parents differ"
        assert np.array_equal(tok[r], ot), f"request {r}: tokens differ"
        assert np.array_equal(sc[r].view(np.int32), osc.view(np.int32)), \
            f"request {r}: scores differ"


def test_select_shared_workspace_across_shapes():
    """One zero-filled workspace serves a sequence of calls of different
    shapes and forms (one-pass, reduction tree, streaming, two passes with wave
    maxima and with summaries, the first two again): each call leaves the
    counters the next one relies on at zero."""
    import torch
    shapes = [(1, 512, SELECT_CODEBOOK, 512, "logsoftmax"), (3, 37, 1001, 300, "ties"),
              (2, 600, 4096, 256, "logsoftmax"), (2, 1024, 4096, 1024, "logsoftmax"),
              (17, 128, SELECT_CODEBOOK, 256, "logsoftmax"), (3, 500, 3001, 200, "special"),
              (1, 64, SELECT_CODEBOOK, 64, "rising"), (2, 256, SELECT_CODEBOOK, 128, "logsoftmax"), (1, 512, SELECT_CODEBOOK, 512, "ties")]
    need = max(ab.onela_select_workspace_bytes(R, P, V, W) for R, P, V, W, _ in shapes)
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    for i, (R, P, V, W, kind) in enumerate(shapes):
        print(f"shared workspace call {i}: R={R} W_prev={P} V={V} W={W} {kind}", flush=True)
        logp, beam = make_select_inputs(R, P, V, 60 + i, kind, True)
        par = torch.empty((R, W), dtype=torch.int32, device="cuda")
        tok = torch.empty((R, W), dtype=torch.int32, device="cuda")
        sc = torch.empty((R, W), dtype=torch.float32, device="cuda")
        ab.onela_select_beams(R, P, V, W, torch.from_numpy(logp).cuda(),
                              torch.from_numpy(beam).cuda(), par, tok, sc, ws, need)
        torch.cuda.synchronize()
        _check(logp, beam, W, par.cpu().numpy(), tok.cpu().numpy(), sc.cpu().numpy())


def _mix(M, m, km):
    """The summary check word's mix (stated beside the one-pass summaries'
    tags): products with odd constants, the second rotated left by 13."""
    a = (M * 0x9E3779B1) & 0xFFFFFFFF
    b = (m * 0x85EBCA77) & 0xFFFFFFFF
    b = ((b << 13) | (b >> 19)) & 0xFFFFFFFF
    return a ^ b ^ ((km * 0xC2B2AE3D) & 0xFFFFFFFF)


@pytest.mark.parametrize("R,P,V,W,form", [(1, 512, SELECT_CODEBOOK, 512, "one_pass"),
                                          (3, 500, 3001, 200, "stream_2_rounds"),
                                          (1, 530, SELECT_CODEBOOK, 200, "stream_2_rounds")])
def test_select_tags_and_epoch_wrap(R, P, V, W, form):
    """The cross-call state of the one-pass and streaming forms in the workspace:
    a call counter (epoch, first word) and, from byte 1024, 8192 16-byte
    summaries (M, m, kM, tag ^ mix).  Planted summaries of an earlier call (older
    tag) with fields that would put the bound above every score, and summaries
    whose check word names this call's tag but whose fields it does not
    match, are not taken; the call matches the oracle and advances the
    epoch.  At the largest tag the epoch starts again at 0 and the region is
    cleared, and the call after it matches too.  Each call's survivor
    counts show that a bound was used (without one every chunk keeps W)."""
    import torch
    from paper_2609_12399_amd.runner import BeamSelector
    sel = BeamSelector(R, P, V, W)
    ws, nsum = sel.workspace, 8192

    def put_u32(off, vals):
        b = torch.from_numpy(np.asarray(vals, dtype=np.uint32).reshape(-1).view(np.uint8).copy())
        ws[off:off + b.numel()].copy_(b)

    def epoch():
        return int(_words(sel, 0, 1)[0])

    def call(seed):
        logp, beam = make_select_inputs(R, P, V, seed, "logsoftmax", True)
        print(f"tagged call seed={seed} epoch={epoch()}", flush=True)
        sel(torch.from_numpy(logp).cuda(), torch.from_numpy(beam).cuda())
        torch.cuda.synchronize()
        _check(logp, beam, W, sel.parents.cpu().numpy(), sel.tokens.cpu().numpy(),
               sel.scores.cpu().numpy())
        kept = _counts(sel)[0].sum(axis=1)
        assert (kept > 0).all() and (kept < 8 * W).all(), kept

    call(89)
    assert _path(sel) == form
    E, top = 5, 0xFFFFFFFF
    put_u32(0, [E])
    planted = np.zeros((nsum, 4), dtype=np.uint32)
    planted[:] = [top, top, 64, E ^ _mix(top, top, 64)]                  # an older call's
    planted[1::2, 3] = (E + 1) ^ _mix(0x1234, top, 64)                   # fields not its own
    put_u32(1024, planted)
    call(90)
    assert epoch() == E + 1
    put_u32(0, [0xFFFFFFFE])
    call(91)
    assert epoch() == 0
    assert int(torch.count_nonzero(ws[1024:1024 + nsum * 16])) == 0
    call(92)
    assert epoch() == 1


@pytest.mark.parametrize("R,P,V,W,kind", [
    (1, 512, SELECT_CODEBOOK, 512, "logsoftmax"), (1, 300, SELECT_CODEBOOK, 64, "ties"),
    (2, 100, SELECT_CODEBOOK, 200, "special"), (4, 64, 65536, 64, "logsoftmax"),
    (3, 500, 3001, 200, "special"), (4, 131, SELECT_CODEBOOK, 33, "ties"),
    (1, 530, SELECT_CODEBOOK, 200, "rising")])
def test_select_waits_that_end_at_once(R, P, V, W, kind):
    """The one-pass and streaming forms wait for other workgroups for a bounded
    time.  With the waits cut to nothing (the shift in the second word of the
    workspace), the bound comes from the summaries that are there at the
    first look, or from none, and most workgroups find no bound: the result
    is the same, in that call and in the next one with the usual waits."""
    import torch
    from paper_2609_12399_amd.runner import BeamSelector
    sel = BeamSelector(R, P, V, W)
    for call, shift in enumerate([63, 63, 0]):
        logp, beam = make_select_inputs(R, P, V, 40 + call, kind, True)
        sel.workspace[4] = shift
        print(f"waits >> {shift} R={R} W_prev={P} V={V} W={W} {kind}", flush=True)
        sel(torch.from_numpy(logp).cuda(), torch.from_numpy(beam).cuda())
        torch.cuda.synchronize()
        _check(logp, beam, W, sel.parents.cpu().numpy(), sel.tokens.cpu().numpy(),
               sel.scores.cpu().numpy())


@pytest.mark.parametrize("R,P,V,W", [(1, 512, SELECT_CODEBOOK, 512), (3, 500, 3001, 200)],
                         ids=["one_pass", "stream"])
def test_select_graph_replays_with_new_scores(R, P, V, W):
    """A selection captured once in a HIP graph and replayed with
    new scores copied into its input buffers between replays (eager work
    and synchronisation in between): every replay matches the oracle."""
    import torch
    from paper_2609_12399_amd.runner import BeamSelector
    logp0, beam0 = make_select_inputs(R, P, V, 70, "logsoftmax", True)
    dl = torch.from_numpy(logp0).cuda()
    db = torch.from_numpy(beam0).cuda()
    s = torch.cuda.Stream()
    sel = BeamSelector(R, P, V, W, stream=s)
    with torch.cuda.stream(s):
        sel(dl, db)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        sel(dl, db)
    torch.cuda.synchronize()
    for rep, kind in enumerate(["logsoftmax", "rising", "logsoftmax", "ties"]):
        logp, beam = make_select_inputs(R, P, V, 80 + rep, kind, True)
        dl.copy_(torch.from_numpy(logp))
        db.copy_(torch.from_numpy(beam))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        print(f"graph replay {rep} ({kind})", flush=True)
        _check(logp, beam, W, sel.parents.cpu().numpy(), sel.tokens.cpu().numpy(),
               sel.scores.cpu().numpy())
