"""The binding keeps the sizes that it checks tensors against: what it refuses
and how must not depend on whether a call asked before.  No GPU: stand-in
tensors, and a host-only plan that the library itself refuses last."""
import pytest

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
