"""The launch a context starts with, and lanes chosen by the caller in whatever order the calls come."""
import pytest

cp = pytest.importorskip("paper_2303_05599_amd")
torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    cp.lib()
    yield


@pytest.mark.parametrize("n,calls,mode", [
    (16384, ("jets",), cp.PUSH_TABLE),
    (16384, ("jets", "lanes"), cp.PUSH_GATHER),
    (16384, ("lanes", "jets"), cp.PUSH_GATHER),
    (16384, ("jets", "table", "lanes"), cp.PUSH_TABLE),
    (16384, ("table", "lanes", "jets"), cp.PUSH_TABLE),
    (39367, ("jets", "lanes"), cp.PUSH_TABLE),      # above 1.5 per site
    (39367, ("lanes",), cp.PUSH_TABLE)])
def test_lanes_and_paths(n, calls, mode):
    ctx = cp.Context(dict(N=162, L_fm=6.0, n_sheets=1, tau_max_fm=0.1), dict(n=n, mass_GeV=1.27))
    for call in calls:
        {"jets": ctx.enable_jets, "lanes": lambda: ctx.set_push_lanes(2), "table": lambda: ctx.set_push_mode(cp.PUSH_TABLE)}[call]()
    assert ctx.push_mode() == mode
    if "lanes" in calls:
        assert ctx.get_launch()["push_lanes"] == 2
    ctx.init_mv()
    ctx.step(3)
    ctx.sync()
    ctx.close()


@pytest.mark.parametrize("N,by", [(384, 4), (432, 4), (486, 4), (512, 8), (576, 4), (1024, 4)])
def test_default_tiles(N, by):
    for prec in (cp.FP64, cp.FP32):
        ctx = cp.Context(dict(N=N, L_fm=6.0, n_sheets=1, tau_max_fm=0.1, precision=prec))
        launch = ctx.get_launch()
        assert (launch["variant"], launch["bx"], launch["by"]) == (3, 64, by)
        ctx.close()
