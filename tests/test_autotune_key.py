"""The key of a stored launch shape tells apart what the timed kernels depend on,
and entries of earlier kernels are not taken up."""
import json
from types import SimpleNamespace

from paper_1611_07289_amd import autotune, pvr, synth


def _plan(n=24, psf=pvr.PVR_PSF_GAUSSIAN, k=3.0, side=16):
    g = synth.iso_grid(n)
    st = [synth.make_stack(synth.grid_center(g), *fr, n, n, 4, (1, 1), 4.0, (1.0, 1.0, 4.0))
          for fr in synth.orthogonal_frames([30.0])]
    P = synth.square_patches(st, side, side)
    dg, ds, dp = pvr.make_descriptors([g], [st], [P])
    return SimpleNamespace(_g=dg, _s=ds, _p=dp, N=sum(p.w * p.h for p in dp), M=P.M, V=n ** 3, P=1,
                           psf=psf, cutoff_k=k,
                           set_tiles=lambda *a: None, set_granules=lambda *a: None)


def test_the_key_depends_on_what_the_kernels_do():
    keys = [autotune.signature(p) for p in (_plan(), _plan(n=25), _plan(side=12), _plan(k=2.5),
                                            _plan(psf=pvr.PVR_PSF_SINC), _plan(psf=pvr.PVR_PSF_SINC, k=2.5))]
    assert len(set(keys)) == len(keys)
    assert autotune.signature(_plan()) == keys[0]


def test_a_choice_timed_on_earlier_kernels_is_not_found(tmp_path):
    key = autotune.signature(_plan())
    db = {v + key.split("-", 1)[1]: {"forward": "tiles/16x16", "adjoint_granule": 1} for v in ("v1-", "v2-")}
    path = tmp_path / "autotune.json"
    path.write_text(json.dumps(db))
    assert key not in autotune._load_cache(str(path))
