"""Training steps in one launch against the same steps as a gradient and an Adam
call each (needs an MI355X): parameters, both moments and the last loss must be
the same bits, since placement depends on the trained surrogate.

Sizes: one point, a whole tile of 16 and one more, the most points held in LDS
(1024) and one more, the largest set; one step, two, a whole launch of 128 and
one more."""
import ctypes

import numpy as np
import pytest

import paper_1105_4840_amd as ppp
from oracle import mlp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# the library's internal launcher (no C entry point trains in one call)
TRAIN = "_ZN3ppp16launch_mlp_trainEPfPKfS2_S2_S2_S2_iS0_S0_S0_fiiP12ihipStream_t"


@pytest.mark.parametrize("n", [1, 16, 17, 300, 1024, 1025, 4096])
@pytest.mark.parametrize("iters", [1, 2, 128, 129])
def test_training_launch_equals_single_steps(n, iters):
    print(f"case mlp train n={n} iters={iters}", flush=True)
    rng = np.random.default_rng(100 * n + iters)
    dev = lambda a: torch.tensor(np.asarray(a, dtype=np.float32), device="cuda")
    data = [dev(a) for a in (rng.uniform(-1, 1, n), rng.normal(size=n), rng.uniform(0, 1, n), rng.normal(size=n),
                             rng.uniform(0, 1, n))]
    P = dev(mlp.init_params(n))
    P2 = P.clone()
    first, lr = 5, 3e-3                  # the moments start as a run in progress would have them
    M, V = dev(rng.normal(size=mlp.NPARAM) * 0.1), dev(np.abs(rng.normal(size=mlp.NPARAM)) * 0.1)
    M2, V2 = M.clone(), V.clone()
    G, L, L2 = torch.zeros_like(P), torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    lib = ppp.lib()
    ptr = ppp._ptr
    for k in range(iters):
        assert lib.ppp_mlp_grad(ptr(P), *[ptr(d) for d in data], n, ptr(G), ptr(L), ppp._stream()) == 0
        assert lib.ppp_mlp_adam(ptr(P), ptr(G), ptr(M), ptr(V), lr, first + k, ppp._stream()) == 0
    train = getattr(lib, TRAIN)
    vp = ctypes.c_void_p
    train.argtypes = [vp] * 6 + [ctypes.c_int] + [vp] * 3 + [ctypes.c_float, ctypes.c_int, ctypes.c_int, vp]
    assert train(ptr(P2), *[ptr(d) for d in data], n, ptr(M2), ptr(V2), ptr(L2), lr, first, iters, ppp._stream()) == 0
    torch.cuda.synchronize()
    for name, a, b in (("parameters", P, P2), ("first moment", M, M2), ("second moment", V, V2), ("loss", L, L2)):
        assert torch.isfinite(a).all(), name
        assert torch.equal(a, b), name
