"""A pooled request that finds no single block for its buffers takes them one by
one: an allocator whose hipMalloc of the block fails, which leaves the runtime's
last error set, as the library's own would.  The request ends with the bits of a
simulation of its own and everything is handed back.  A simulation that finds no
memory leaves no error for the next."""
import ctypes

import numpy as np
import pytest

from tests import harness as H

pytestmark = pytest.mark.gpu


def _hip():
    """The HIP runtime that this process has loaded."""
    with open("/proc/self/maps") as m:
        path = next(l.split()[-1] for l in m if "libamdhip64.so" in l)
    return ctypes.CDLL(path)


class NoBlocks:
    """lbl_env callbacks: hipMalloc, but for anything above `limit` bytes of a
    size that no device has."""

    def __init__(self, limit):
        from paper_1104_0078_amd import lbl
        import torch
        torch.cuda.init()
        torch.cuda.current_stream().synchronize()
        self.lbl, self.live, self.refused = lbl, set(), 0
        lbl.library()
        hip = _hip()

        def _alloc(ctx, nbytes, stream):
            ptr = ctypes.c_void_p()
            size = nbytes if nbytes <= limit else 1 << 50
            if hip.hipMalloc(ctypes.byref(ptr), ctypes.c_size_t(size)) != 0:
                self.refused += 1
                return None
            self.live.add(ptr.value)
            return ptr.value

        def _free(ctx, ptr, stream):
            self.live.discard(ptr)
            hip.hipFree(ctypes.c_void_p(ptr))

        self._alloc, self._free = lbl.ALLOC_FN(_alloc), lbl.FREE_FN(_free)

    def env(self):
        e = self.lbl.lbl_env()
        e.device, e.stream, e.ctx = 0, None, None
        e.alloc, e.free = self._alloc, self._free
        return e


@pytest.mark.parametrize("lattice,shape", [(H.D2Q9, (32, 24, 1)), (H.D3Q19, (12, 9, 7))])
@pytest.mark.parametrize("user", [False, True])
def test_request_without_a_block(lattice, shape, user):
    from paper_1104_0078_amd import lbl
    c = H.config(lattice=lattice, smol=H.FV, shape=shape, a=-0.04, b=0.04)
    print("pool without blocks:", lattice, shape, "user", user, flush=True)
    ini = lbl.make_init(psi_std=1e-3)
    with lbl.Sim(H.lbl_params(c), ini) as sim:
        if user:
            ini = lbl.make_init(lbl.LBL_INIT_USER, f0=sim.observe(lbl.LBL_OBS_POP),
                                psi0=sim.observe(lbl.LBL_OBS_PSI))
        sim.step(6)
        psi = sim.observe(lbl.LBL_OBS_PSI)
    n = shape[0] * shape[1] * shape[2]
    mem = NoBlocks(8 * n * (lattice + 1))  # the largest single buffer, and staged states
    with lbl.Pool(1 << 30, memory=mem) as pool:
        rid = pool.submit(H.lbl_params(c), ini, 6, keep_psi=True)
        while pool.run(4) > 0:
            pass
        assert mem.refused == 1
        assert pool.poll(rid) == (lbl.LBL_REQ_DONE, 6)
        np.testing.assert_array_equal(pool.result(rid, lbl.LBL_RES_PSI), psi)
    assert not mem.live


def test_no_error_is_left_for_the_next_simulation():
    from paper_1104_0078_amd import lbl
    c = H.config(lattice=H.D2Q9, smol=H.FV, shape=(32, 24, 1))
    mem = NoBlocks(0)
    with pytest.raises(lbl.LblError) as e:
        lbl.Sim(H.lbl_params(c), lbl.make_init(psi_std=1e-3), memory=mem)
    assert e.value.code == lbl.LBL_E_NOMEM
    assert mem.refused and not mem.live
    with lbl.Sim(H.lbl_params(c), lbl.make_init(psi_std=1e-3)) as sim:
        sim.step(2)
        assert np.isfinite(sim.observe(lbl.LBL_OBS_PSI)).all()
