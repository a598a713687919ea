"""Exponentials at the ends of the range of rates: a draw is -log(u) times the
reciprocal of the rate, each rounded once, also where the reciprocal is subnormal
(rates above 2^1022) or infinite (below 2^-1024).  Exact: -log(u) comes from rate
1, and numpy's product has the same single rounding.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2201_06604_amd as P  # noqa: E402

RATES = [3e-309, 5.6e-309, 2.0 ** -1022, 0.75, 2.0 ** 1022, 7.362967829554601e307, 1.4704137154461813e308,
         1.732337106235814e308, np.finfo(np.float64).max]
S, DRAWS = 129, 64


def plain(s, n, rate, gen, cfg):
    return P.mrg_generate(s, n, P.MRG_EXPONENTIAL, P.MRG_F64, rate, gen=gen, cfg=cfg)


def paper(s, n, rate, gen, cfg):
    out = torch.zeros((n // 100, 100), dtype=torch.float64, device="cuda")
    P.mrg_generate_paper(s, n // 100, 100, 8, 16, P.MRG_EXPONENTIAL, P.MRG_F64, rate, out=out, gen=gen)
    return out


def batch(s, n, rate, gen, cfg):
    out = torch.zeros(n, dtype=torch.float64, device="cuda")
    plan = P.BatchPlan([P.make_request(s, n, P.MRG_EXPONENTIAL, P.MRG_F64, rate, out)], cfg=cfg)
    plan.upload()
    plan.launch()
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("call,gen,cfg", [
    (plain, P.MRG_GEN_MRG32K3A, None), (plain, P.MRG_GEN_MRG31K3P, None),
    (plain, P.MRG_GEN_MRG32K3A, dict(arith=1, block=256, chunk=7)), (paper, P.MRG_GEN_MRG32K3A, None),
    (paper, P.MRG_GEN_MRG31K3P, None), (batch, P.MRG_GEN_MRG32K3A, None),
    (batch, P.MRG_GEN_MRG32K3A, dict(gang_waves=1)), (batch, P.MRG_GEN_MRG32K3A, dict(wide_stores=2))], ids=str)
def test_a_draw_is_minus_log_u_times_the_reciprocal(call, gen, cfg):
    n = S * DRAWS // 100 * 100

    def draws(rate):
        s = P.mrg_streams_create_device(P.mrg_creator_init([12345] * 6, gen=gen), S, gen=gen)
        return call(s, n, rate, gen, cfg).cpu().numpy().ravel()[:n]
    log = draws(1.0)
    for rate in RATES:
        with np.errstate(over="ignore", under="ignore"):
            want = log * (np.float64(1.0) / np.float64(rate))
        np.testing.assert_array_equal(draws(rate), want, err_msg=str(rate))
