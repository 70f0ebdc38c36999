"""The binding keeps the sizes that it checks tensors against: what it refuses
and how must not depend on whether a call asked before.  No GPU: stand-in
tensors, and a host-only plan that the library itself refuses last."""
import numpy as np
import pytest
import torch

from paper_2607_04749_amd import etc
from paper_2607_04749_amd.workloads import TINY_GPT, Parallel as P


class Buffer:
    """What the binding looks at in a tensor."""

    def __init__(self, nbytes, gpu=True, contiguous=True):
        self.nbytes, self.is_cuda, self._contiguous = nbytes, gpu, contiguous

    def is_contiguous(self):
        return self._contiguous

    def numel(self):
        return self.nbytes

    def element_size(self):
        return 1

    def data_ptr(self):
        return 4096


def _plan():
    return etc.etc_plan(TINY_GPT, P(2, 2, 1), P(4, 1, 1),
                        flags=etc.PLAN_HOST_ONLY | etc.PLAN_SKETCH | etc.PLAN_DIRECT_REFER)


@pytest.mark.parametrize("asked_before", [False, True])
def test_same_checks_on_every_call(asked_before):
    plan = _plan()
    d = 1
    h = int(plan.pairing()[d])
    src = [Buffer(n) for n in plan.arena_bytes(etc.SIDE_SRC, h)]
    dst = [Buffer(n) for n in plan.arena_bytes(etc.SIDE_DST, d)]
    total = plan.send_layout(h)[3]
    sizes = [int(plan.send_layout(s)[1][d]) for s in range(plan.S)]
    chunk = [int(plan.chunk_layout(s, 2)[0][d]) for s in range(plan.S)]
    s = next(i for i, n in enumerate(sizes) if n)

    def msgs(per, short=0, **kw):
        return [Buffer(n - (short if i == s else 0), **kw) if n else None for i, n in enumerate(per)]

    def short(arenas, k):
        return [Buffer(b.nbytes - (i == k)) for i, b in enumerate(arenas)]

    def calls():
        yield lambda: etc.etc_pack(plan, h, src, Buffer(total), 0), None
        yield lambda: etc.etc_refer(plan, d, src, dst, 0), None
        yield lambda: etc.etc_unpack(plan, d, msgs(sizes), dst, 0), None
        yield lambda: etc.etc_unpack_kind(plan, d, 2, msgs(chunk), dst[2], 0), None
        yield lambda: etc.etc_pack_kind(plan, h, 0, src[0], Buffer(plan.chunk_layout(h, 0)[2]), 0), None
        yield (lambda: etc.etc_pack(plan, h, src, Buffer(total - 1), 0),
               f"send_buf holds {total - 1} bytes; the plan needs {total}")
        yield (lambda: etc.etc_pack(plan, h, short(src, 3), Buffer(total), 0),
               rf"src_arenas\[3\] holds {src[3].nbytes - 1} bytes; the plan needs {src[3].nbytes}")
        yield (lambda: etc.etc_refer(plan, d, src, short(dst, 0), 0), rf"dst_arenas\[0\] holds {dst[0].nbytes - 1} ")
        yield (lambda: etc.etc_unpack(plan, d, msgs(sizes, 1), dst, 0),
               rf"msgs\[{s}\] holds {sizes[s] - 1} bytes; the plan needs {sizes[s]}")
        yield (lambda: etc.etc_unpack_kind(plan, d, 2, msgs(chunk, 1), dst[2], 0),
               rf"msgs\[{s}\] holds {chunk[s] - 1} bytes; the plan needs {chunk[s]}")
        yield lambda: etc.etc_unpack(plan, d, msgs(sizes, gpu=False), dst, 0), "must be a contiguous GPU tensor"
        yield lambda: etc.etc_unpack(plan, d, msgs(sizes, contiguous=False), dst, 0), "must be a contiguous GPU tensor"

    for _ in range(1 + asked_before):
        for call, refused in calls():
            if refused:
                with pytest.raises(ValueError, match=refused):
                    call()
            else:
                with pytest.raises(etc.EtcError, match="HOST_ONLY"):
                    call()
    with pytest.raises(etc.EtcError):
        etc.etc_pack(plan, plan.S, src, Buffer(total), 0)
    plan.free()
    for call, _ in calls():
        with pytest.raises(ValueError, match="plan was freed"):
            call()


def _steps(plan, s, d):
    """Every device call of the binding, (name, call(rank, kind)), with buffers
    that fit source rank s, target rank d and kind 0 exactly."""
    h = int(plan.pairing()[d])
    src = [Buffer(n) for n in plan.arena_bytes(etc.SIDE_SRC, s)]
    home = [Buffer(n) for n in plan.arena_bytes(etc.SIDE_SRC, h)]
    dst = [Buffer(n) for n in plan.arena_bytes(etc.SIDE_DST, d)]
    send = Buffer(plan.send_layout(s)[3])
    msgs = [Buffer(int(plan.send_layout(x)[1][d])) for x in range(plan.S)]
    chunk = Buffer(plan.chunk_layout(s, 0)[2])
    parts = [Buffer(int(plan.chunk_layout(x, 0)[0][d])) for x in range(plan.S)]
    return [
        ("src", lambda r, k: etc.etc_pack(plan, r, src, send, 0)),
        ("dst", lambda r, k: etc.etc_unpack(plan, r, msgs, dst, 0)),
        ("dst", lambda r, k: etc.etc_refer(plan, r, home, dst, 0)),
        ("src kind", lambda r, k: etc.etc_pack_kind(plan, r, k, src[0], chunk, 0)),
        ("dst kind", lambda r, k: etc.etc_unpack_kind(plan, r, k, parts, dst[0], 0)),
        ("dst kind", lambda r, k: etc.etc_refer_kind(plan, r, k, home[0], dst[0], 0)),
    ]


def _two_stage_plan():
    return etc.etc_plan(TINY_GPT, P(2, 2, 1), P(1, 2, 1),
                        flags=etc.PLAN_HOST_ONLY | etc.PLAN_SKETCH | etc.PLAN_DIRECT_REFER)


def _by_size(plan, side, n):
    return sorted(range(n), key=lambda r: plan.arena_elems(side, r))


@pytest.mark.parametrize("step", range(6))
def test_a_rank_changed_in_place_is_checked_anew(step):
    """A rank or kind may be any integer that ctypes takes, a 0-d tensor among
    them: one that the caller changes is another rank, with sizes of its own."""
    plan = _two_stage_plan()
    src, dst = _by_size(plan, etc.SIDE_SRC, plan.S), _by_size(plan, etc.SIDE_DST, plan.D)
    assert plan.arena_elems(etc.SIDE_SRC, src[0]) < plan.arena_elems(etc.SIDE_SRC, src[-1])
    assert plan.arena_elems(etc.SIDE_DST, dst[0]) < plan.arena_elems(etc.SIDE_DST, dst[-1])
    what, call = _steps(plan, src[0], dst[0])[step]
    ranks = src if "src" in what else dst
    rank, kind = torch.tensor(ranks[0]), torch.tensor(0)
    with pytest.raises(etc.EtcError, match="HOST_ONLY"):
        call(rank, kind)
    rank.fill_(ranks[-1])
    with pytest.raises(ValueError, match="the plan needs"):
        call(rank, kind)
    if "kind" in what:
        rank.fill_(ranks[0])
        with pytest.raises(etc.EtcError, match="HOST_ONLY"):
            call(rank, kind)
        kind += 1
        with pytest.raises(ValueError, match="the plan needs"):
            call(rank, kind)


@pytest.mark.parametrize("step", range(6))
@pytest.mark.parametrize("as_int", [int, np.int32, np.uint64, np.array, torch.tensor])
def test_a_rank_of_any_integer_type_is_taken(step, as_int):
    plan = _two_stage_plan()
    what, call = _steps(plan, 1, 1)[step]
    for _ in range(2):
        with pytest.raises(etc.EtcError, match="HOST_ONLY"):
            call(as_int(1), as_int(0))
    with pytest.raises(etc.EtcError):
        call(as_int(1000), as_int(0))
    if "kind" in what:
        with pytest.raises(etc.EtcError):
            call(as_int(1), as_int(4))
    assert len(getattr(plan, "_sizes", ())) < 16
