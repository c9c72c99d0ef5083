"""What a user of the rasterizer has it do, as cases that can be timed and compared.

Each case is one pass through the package's public entry points over inputs drawn on the GPU from a
seed alone: rendering, a render with its gradients, the training steps built from them, the anchor
decoder, the photometric loss and the densification event. Sizes are those of the package's own
benchmark, fits and tests, with odd ones between them.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs, and the buffers a program keeps between calls
    run(state)           one pass; its outputs
    work(case)           bytes and operations of one pass that it cannot do without
    exact(case, seed)    the outputs in 64 bits by plain torch, where that is quick
"""
from __future__ import annotations

import math

import torch

from paper_2601_19489_amd import _lib, scenes
from paper_2601_19489_amd.anchors import MLP_NAMES, AnchorDecoder
from paper_2601_19489_amd.batched import BatchedRasterizer, TrainStep
from paper_2601_19489_amd.rasterizer import PARAM_NAMES, Adam, Rasterizer, l1_loss

# learning rates of the package's fits and benchmark
LRS = dict(means=1.6e-4, log_scales=5e-3, quats=1e-3, opacity_logits=5e-2, sh=2.5e-3)
ANCHOR_LRS = dict(feat=5e-3, offsets=1e-2, scaling=1e-4, w1=2e-3, b1=2e-3, w2=2e-3, b2=2e-3)
GROW_VIEWS = 3      # views of a densification event
RADIUS = 4.0        # camera distance from the scene's centre


def listed():
    return [
        # the smallest call: a render with its gradients where launches and latency are the time
        dict(name='raster_tiny', kind='raster', scene='cloud', n=1000, w=64, h=64, deg=0, tile=16,
             depth=False, inverse=False),
        # the small anchor-vs-plain fit's view: 20k Gaussians at 192 x 192
        dict(name='raster_20k', kind='raster', scene='surface', n=20_000, w=192, h=192, deg=0,
             tile=16, depth=False, inverse=False),
        # ragged sizes, disparity supervision: colour and depth gradients of a trained-like scene
        dict(name='raster_odd', kind='raster', scene='fit', n=123_457, w=1277, h=719, deg=2,
             tile=16, depth=True, inverse=True),
        # viewing a finished scene: forward only
        dict(name='render_1080p', kind='render', scene='surface', n=1_000_000, w=1920, h=1080,
             deg=3, tile=16, depth=False, inverse=False),
        # the training step of the benchmark: forward, L1, backward fused with Adam
        dict(name='step_1m', kind='step', scene='surface', n=1_000_000, w=1600, h=1066, deg=3,
             tile=16, depth=False, inverse=False),
        # the densifying fit's step near its start: Eq. 5 loss, depth loss, backward, Adam
        dict(name='fit_300k', kind='fit', scene='fit', n=300_000, w=1600, h=1066, deg=3, tile=16,
             depth=True, inverse=False),
        # a minibatch of views of mixed resolutions, replayed from its graph
        dict(name='views_8', kind='views', scene='surface', n=1_000_000, views=8, scale=1.0, deg=3,
             tile=16),
        # the anchor decoder alone, forward and backward: the small fit's and the benchmark's size
        dict(name='decode_2k', kind='decode', anchors=2000),
        dict(name='decode_100k', kind='decode', anchors=100_000),
        # the anchor form's whole training step (direct colours, 10 children per anchor)
        dict(name='anchor_100k', kind='anchor', anchors=100_000, w=1600, h=1066, tile=16),
        # the Eq. 5 loss and its gradient on one view
        dict(name='photo_1600', kind='photo', w=1600, h=1066),
        # a densification event: masks, scores, threshold, plan, growth of parameters and moments
        dict(name='grow_1m', kind='grow', scene='fit', n=1_000_000, w=1600, h=1066, deg=3,
             tile=16),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(['raster', 'raster', 'raster', 'render', 'step', 'step', 'fit', 'fit',
                       'views', 'decode', 'anchor', 'photo', 'grow'])
    w = logint(48, 1920)
    h = max(40, min(1080, int(w * rng.uniform(0.5, 1.0))))
    tile = rng.choice([16, 16, 16, 16, 8, 32])
    # up to two Gaussians a pixel: more than any of the benchmark's scenes and fits has
    n = logint(300, min(1_000_000, 2 * w * h))
    if kind == 'decode':
        return dict(kind=kind, anchors=logint(50, 200_000))
    if kind == 'photo':
        return dict(kind=kind, w=w, h=h)
    if kind == 'anchor':
        return dict(kind=kind, anchors=logint(100, min(100_000, w * h // 5)), w=w, h=h, tile=tile)
    if kind == 'views':
        scale = round(w / 1920, 3)      # of the benchmark's resolutions, 960 x 540 the smallest
        return dict(kind=kind, scene='surface', n=min(n, max(300, int(1e6 * scale * scale))),
                    views=rng.randint(2, 8), scale=scale, deg=rng.randint(0, 3), tile=tile)
    scene = 'fit' if kind in ('fit', 'grow') else rng.choice(['cloud', 'surface', 'fit'])
    c = dict(kind=kind, scene=scene, n=n, w=w, h=h, deg=rng.randint(0, 3), tile=tile)
    if kind != 'grow':
        c.update(depth=kind == 'fit' or (kind == 'raster' and rng.random() < 0.4),
                 inverse=rng.random() < 0.25)
    return c


# -- inputs ------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device='cuda').manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device='cuda')


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device='cuda')


def _surface_points(g, n):
    """Points of 3 unit planes and 4 spheres with N(0, 0.01^2) noise."""
    surf = torch.randint(0, 7, (n,), generator=g, device='cuda')
    pos = 2.0 * _rand(g, 3, n) - 1.0
    sdir = _randn(g, 3, n)
    sdir /= sdir.norm(dim=0, keepdim=True).clamp_min(1e-6)
    for k, (axis, off) in enumerate(scenes._PLANES):
        pos[axis] = torch.where(surf == k, torch.full_like(pos[axis], off), pos[axis])
    for k, (centre, radius) in enumerate(scenes._SPHERES):
        c = torch.tensor(centre, device='cuda')[:, None]
        pos = torch.where(surf == 3 + k, c + radius * sdir, pos)
    return pos + 0.01 * _randn(g, 3, n)


def _scene(g, scene, n, deg):
    """Gaussian parameters: the uniform cloud, the heavy-tailed surface cloud, or a scene as a fit
    has it, where a Gaussian is about as large as the distance to its neighbours."""
    if scene == 'cloud':
        means = 2.0 * _rand(g, 3, n) - 1.0
        ls = -3.0 + 0.5 * _randn(g, 3, n)
    else:
        means = _surface_points(g, n)
        if scene == 'surface':
            large = (_rand(g, 1, n) < 0.1).float()
            ls = -4.0 + 2.5 * large + 0.5 * _randn(g, 3, n)
        else:
            spacing = math.sqrt(17.0 / n)   # about 17 square units of surface
            ls = math.log(spacing) + 0.4 * _randn(g, 3, n)
    q = _randn(g, 4, n)
    K = (deg + 1) ** 2
    sh = 0.1 * _randn(g, K, 3, n)
    sh[0] = (_rand(g, 3, n) - 0.5) * (2.0 * math.sqrt(math.pi))
    return dict(means=means.contiguous(), log_scales=ls.contiguous(),
                quats=(q / q.norm(dim=0, keepdim=True).clamp_min(1e-6)).contiguous(),
                opacity_logits=_randn(g, n), sh=sh)


def _moved(g, p):
    """The scene as it is in the middle of a fit of it: near the scene its targets were made of."""
    step = dict(means=0.002, log_scales=0.1, quats=0.05, opacity_logits=0.3, sh=0.05)
    return {k: v + step[k] * torch.randn(v.shape, generator=g, device='cuda') for k, v in p.items()}


def _orbit(g, count, sizes, tile, inverse=False):
    """Cameras around the scene, a direction each."""
    a = _rand(g, count, 2).cpu().tolist()
    cams = []
    for (x, y), (w, h) in zip(a, sizes):
        az, el = 2.0 * math.pi * x, 0.4 * y - 0.2
        eye = (RADIUS * math.sin(az) * math.cos(el), -RADIUS * math.sin(el),
               -RADIUS * math.cos(az) * math.cos(el))
        c = scenes.look_at_camera(eye, (0.0, 0.0, 0.0), w, h, tile=tile)
        c.depth_mode = 1 if inverse else 0
        cams.append(c)
    return cams


def _adam(p, lrs):
    """Adam with the moments and the step count of a fit under way."""
    opt = Adam(p, lrs)
    for v in opt.v.values():
        v.fill_(1e-14)
    opt.step_count.fill_(500)
    return opt


def _raster_for(case, cam, n, p, deg, deferred=False):
    """A rasterizer with its pair buffers sized, as a program has after its first frame."""
    R = Rasterizer(n, cam, deg, headroom=1.5, deferred=deferred)
    R.forward(p)
    return R


def _views_sizes(case):
    s = case['scale']
    return [(max(40, int(w * s)), max(40, int(h * s)))
            for w, h in scenes.ORBIT_RESOLUTIONS[:case['views']]]


def _trained(opt, loss):
    return dict(params=opt.params, m=opt.m, v=opt.v, loss=loss)


def _anchors(g, A):
    """Anchors and the shared decoder, spread as the package's generators spread them."""
    a = dict(feat=0.1 * _randn(g, 32, A), pos=_surface_points(g, A) + 0.02 * _randn(g, 3, A),
             offsets=0.5 * _randn(g, 30, A),
             scaling=torch.exp(math.log(0.02) + 0.3 * _randn(g, 6, A)))
    bi, bh = 1.0 / math.sqrt(35), 1.0 / math.sqrt(32)
    m = dict(w1=bi * (2 * _rand(g, 96, 35) - 1), b1=bi * (2 * _rand(g, 96) - 1),
             w2=bh * (2 * _rand(g, 110, 32) - 1), b2=bh * (2 * _rand(g, 110) - 1))
    return {k: v.contiguous() for k, v in a.items()}, m


def _smooth_image(g, h, w):
    """An image in [0, 1] with the low-frequency look of a photograph, and some grain."""
    low = _rand(g, 1, 3, max(2, h // 32), max(2, w // 32))
    up = torch.nn.functional.interpolate(low, size=(h, w), mode='bilinear', align_corners=False)[0]
    return (up + 0.05 * _randn(g, 3, h, w)).clamp(0.0, 1.0).contiguous()


# -- the cases ----------------------------------------------------------------

def prepare(case, seed):
    g = _gen(seed)
    kind = case['kind']
    s = dict(case=dict(case), kind=kind)
    if kind == 'photo':
        h, w = case['h'], case['w']
        tgt = _smooth_image(g, h, w)
        s.update(tgt=tgt, img=(tgt + 0.05 * _randn(g, 3, h, w)).clamp(0.0, 1.0).contiguous(),
                 loss=torch.zeros(3, device='cuda'), dI=torch.empty((3, h, w), device='cuda'),
                 ws=torch.empty(_lib.gs_photo_loss_workspace(3, h, w), dtype=torch.uint8,
                                device='cuda'))
        return s
    if kind == 'decode':
        A = case['anchors']
        a, m = _anchors(g, A)
        cam = _orbit(g, 1, [(1600, 1066)], 16)[0]
        dec = AnchorDecoder(A)
        dchild = {k: _randn(g, *v.shape) for k, v in dec.children.items()}
        s.update(a=a, m=m, cam=_lib.camera(cam), dec=dec, dchild=dchild,
                 da={k: torch.empty_like(a[k]) for k in ('feat', 'offsets', 'scaling')},
                 dm={k: torch.empty_like(m[k]) for k in MLP_NAMES})
        return s
    if kind == 'anchor':
        A = case['anchors']
        a, m = _anchors(g, A)
        cam = _orbit(g, 1, [(case['w'], case['h'])], case['tile'])[0]
        dec = AnchorDecoder(A)
        R = _raster_for(case, cam, dec.N, dec.decode(a, m, _lib.camera(cam)), _lib.GS_DIRECT)
        target = R.image.clone()
        a['feat'] += 0.05 * _randn(g, 32, A)
        train = dict(feat=a['feat'], offsets=a['offsets'], scaling=a['scaling'], **m)
        s.update(a=a, m=m, dec=dec, R=R, target=target, opt=_adam(train, ANCHOR_LRS),
                 grads={k: torch.empty_like(v) for k, v in train.items()},
                 dchild={k: torch.empty_like(v) for k, v in dec.children.items()},
                 dI=torch.empty_like(R.image), loss=torch.zeros(1, device='cuda'))
        return s
    n, deg, tile = case['n'], case['deg'], case['tile']
    truth = _scene(g, case['scene'], n, deg)
    if kind == 'views':
        sizes = _views_sizes(case)
        B = BatchedRasterizer(n, _orbit(g, len(sizes), sizes, tile), deg, tile=tile, headroom=1.5,
                              deferred=True)
        B.size_pairs(truth)
        B.forward(truth)
        st = TrainStep(B, _moved(g, truth), [b['image'].clone() for b in B.buf], LRS)
        for v in st.v.values():
            v.fill_(1e-14)
        st.step_count.fill_(500)
        st.run()
        st.check_capacity()
        st.capture()
        s.update(st=st)
        return s
    inverse = case.get('inverse', False)
    w, h = case['w'], case['h']
    if kind == 'grow':
        cams = _orbit(g, GROW_VIEWS, [(w, h)] * GROW_VIEWS, tile)
        R = _raster_for(case, cams[0], n, truth, deg)
        gcams = [_lib.camera(c) for c in cams]
        targets = []
        for c in gcams:
            R.cam = c
            R.forward(truth)
            targets.append(R.image.clone())
        p = _moved(g, truth)
        opt = _adam(p, LRS)
        for k in PARAM_NAMES:
            opt.m[k] += 1e-8 * torch.randn(p[k].shape, generator=g, device='cuda')
        dev = dict(device='cuda')
        # room for the largest outcome (every Gaussian twice), for parameters and both moments
        room = [{k: torch.zeros(2 * v.numel(), **dev) for k, v in p.items()} for _ in range(3)]
        s.update(room=room, R=R, cams=gcams, targets=targets, p=p, opt=opt, eps=_randn(g, 2, 3, n),
                 score=torch.empty(n, dtype=torch.int32, **dev),
                 count=torch.empty(n, dtype=torch.int32, **dev),
                 prune=torch.empty(n, dtype=torch.float64, **dev),
                 photo=torch.zeros(GROW_VIEWS, 3, **dev),
                 photo_ws=torch.empty(_lib.gs_photo_loss_workspace(3, h, w), dtype=torch.uint8,
                                      **dev),
                 mask=torch.empty(h * w, dtype=torch.uint8, **dev),
                 minmax=torch.empty(2, dtype=torch.int32, **dev),
                 hist=torch.empty(_lib.SCORE_BINS, dtype=torch.int32, **dev),
                 thr=torch.zeros(1, dtype=torch.int32, **dev),
                 n_out=torch.zeros(1, dtype=torch.int32, **dev),
                 ws=torch.empty(_lib.gs_densify_workspace(n), dtype=torch.uint8, **dev))
        return s
    cam = _orbit(g, 1, [(w, h)], tile, inverse)[0]
    s.update(cam=cam)
    if kind == 'render':
        s.update(p=truth, R=_raster_for(case, cam, n, truth, deg))
    elif kind == 'raster':
        R = _raster_for(case, cam, n, truth, deg)
        s.update(p=truth, R=R, grads={k: torch.empty_like(v) for k, v in truth.items()},
                 dI=_randn(g, 3, h, w) / (3 * h * w),
                 dD=0.1 * _randn(g, h, w) / (h * w) if case['depth'] else None)
    else:
        R = _raster_for(case, cam, n, truth, deg, deferred=kind == 'step')
        target, depth = R.image.clone(), R.depth.clone()
        p = _moved(g, truth)
        s.update(p=p, R=R, target=target, opt=_adam(p, LRS), dI=torch.empty_like(R.image),
                 loss=torch.zeros(1, device='cuda'))
        if kind == 'fit':
            s.update(depth=(depth * (1.0 + 0.01 * _randn(g, h, w))).contiguous(),
                     dD=torch.empty_like(depth), photo=torch.zeros(3, device='cuda'),
                     ws=torch.empty(_lib.gs_photo_loss_workspace(3, h, w), dtype=torch.uint8,
                                    device='cuda'),
                     grads={k: torch.empty_like(v) for k, v in p.items()})
    return s


def run(s):
    kind = s['kind']
    if kind == 'photo':
        _, h, w = s['img'].shape
        _lib.gs_photo_loss(s['img'], s['tgt'], 3, h, w, 0.2, s['ws'], s['loss'], s['dI'])
        return dict(loss=s['loss'], dI=s['dI'])
    if kind == 'decode':
        ch = s['dec'].decode(s['a'], s['m'], s['cam'])
        s['dec'].backward(s['a'], s['m'], s['cam'], s['dchild'], s['da'], s['dm'])
        return dict(children=ch, danchors=s['da'], dmlp=s['dm'])
    if kind == 'anchor':
        R, dec = s['R'], s['dec']
        ch = dec.decode(s['a'], s['m'], R.cam)
        R.forward(ch)
        l1_loss(R.image, s['target'], s['dI'], s['loss'])
        R.backward(ch, s['dI'], None, s['dchild'])
        gr = s['grads']
        dec.backward(s['a'], s['m'], R.cam, s['dchild'],
                     {k: gr[k] for k in ('feat', 'offsets', 'scaling')},
                     {k: gr[k] for k in MLP_NAMES})
        s['opt'].step(gr)
        return dict(grads=gr, **_trained(s['opt'], s['loss']))
    if kind == 'views':
        st = s['st']
        st.replay()
        return dict(params=st.p, m=st.m, v=st.v, loss=st.loss)
    R, p = s['R'], s['p']
    if kind == 'render':
        image, depth = R.forward(p)
        return dict(image=image, depth=depth)
    if kind == 'raster':
        image, depth = R.forward(p)
        grads = R.backward(p, s['dI'], s['dD'], s['grads'])
        return dict(image=image, depth=depth, grads=grads)
    if kind == 'step':
        R.forward(p, check_overflow=False)
        l1_loss(R.image, s['target'], s['dI'], s['loss'])
        R.backward_adam(p, s['dI'], s['opt'])
        return _trained(s['opt'], s['loss'])
    c = s['case']
    if kind == 'fit':
        R.forward(p)
        _lib.gs_photo_loss(R.image, s['target'], 3, c['h'], c['w'], 0.2, s['ws'], s['photo'],
                           s['dI'])
        s['loss'].zero_()
        _lib.gs_depth_l1_loss(R.depth, s['depth'], c['h'] * c['w'], 0.05, s['dD'], s['loss'])
        R.backward(p, s['dI'], s['dD'], s['grads'])
        s['opt'].step(s['grads'])
        return dict(photo=s['photo'], **_trained(s['opt'], s['loss']))
    return _grow(s)


def _grow(s):
    """One densification event, as the densifying fit makes it."""
    c, R, p, n = s['case'], s['R'], s['p'], s['case']['n']
    hw = c['h'] * c['w']
    s['score'].zero_()
    s['prune'].zero_()
    for v, (cam, target) in enumerate(zip(s['cams'], s['targets'])):
        R.cam = cam
        R.forward(p)
        photo = s['photo'][v]
        _lib.gs_error_mask(R.image, target, hw, 0.1, s['mask'], s['minmax'])
        _lib.gs_photo_loss(R.image, target, 3, c['h'], c['w'], 0.2, s['photo_ws'], photo, None)
        s['count'].zero_()
        _lib.gs_split_score(R.splats, n, R.vals, R.ranges, R.cam, s['mask'], s['count'])
        _lib.gs_prune_accumulate(s['count'], n, photo, s['prune'], s['score'])
    _lib.gs_densify_threshold(s['score'], n, 2 * GROW_VIEWS, n // 3, s['hist'], s['thr'])
    thr = int(s['thr'].item()) & 0xFFFFFFFF
    _lib.gs_densify_prune_plan(s['score'], p['log_scales'], n, thr, 0.02, s['prune'], 0.9,
                               s['ws'], s['n_out'])
    n_out = int(s['n_out'].item()) & 0xFFFFFFFF
    for old, moments, room in zip((p, s['opt'].m, s['opt'].v), (False, True, True), s['room']):
        new = {k: room[k][:v.numel() // n * n_out].view(v.shape[:-1] + (n_out,))
               for k, v in old.items()}
        _lib.gs_densify_apply(_lib.gaussians(*[old[k] for k in PARAM_NAMES]), n, c['deg'],
                              None if moments else s['eps'], s['ws'], n_out, moments,
                              _lib.gaussians(*[new[k] for k in PARAM_NAMES]))
    return dict(score=s['score'], photo=s['photo'], threshold=thr, n_out=n_out, new=s['room'])


# -- work ---------------------------------------------------------------------

def _blended(scene, n, pixels, width):
    """About how many splats a pixel composites before it is opaque or out of splats."""
    f = width / (2.0 * math.tan(math.radians(30.0))) / RADIUS   # pixels per unit of the scene
    if scene == 'cloud':
        area = 25.0 * math.exp(2 * -3.0 + 0.5) * f * f
    elif scene == 'surface':
        area = 25.0 * (0.9 * math.exp(-8.0 + 0.5) + 0.1 * math.exp(-3.0 + 0.5)) * f * f
    else:
        area = 25.0 * (17.0 / n) * f * f
    return min(160.0, n * min(area, pixels) / pixels)


def _params(deg):
    return 11 + 3 * (deg + 1) ** 2 if deg >= 0 else 14


def work(case):
    kind = case['kind']
    # operations of one (pixel, splat) evaluation, forward and backward
    fwd, bwd = 30.0, 60.0
    if kind == 'photo':
        px = case['w'] * case['h']
        # two images read, one gradient written; 5 forward and 3 backward window sums, 22 taps each
        return dict(bytes=36.0 * px, flops=3.0 * px * 8 * 22 * 2)
    if kind in ('decode', 'anchor'):
        A = case['anchors']
        if kind == 'decode':
            # 71 anchor values read twice, 14 values a child written and as many gradients read,
            # 68 gradient values written
            mac = 96 * 35 + 110 * 32
            return dict(bytes=4.0 * A * (2 * 71 + 280 + 68), flops=2.0 * A * mac * 4)
        px = case['w'] * case['h']
        ev = px * _blended('surface', 10 * A, px, case['w'])
        return dict(bytes=4.0 * A * (71 + 6 * 68) + 24.0 * px, flops=ev * (fwd + bwd))
    n, P = case['n'], _params(case['deg'])
    if kind == 'views':
        px = sum(w * h for w, h in _views_sizes(case))
        ev = sum(w * h * _blended(case['scene'], n, w * h, w) for w, h in _views_sizes(case))
        return dict(bytes=24.0 * n * P + 12.0 * px, flops=ev * (fwd + bwd))
    px = case['w'] * case['h']
    ev = px * _blended(case['scene'], n, px, case['w'])
    if kind == 'render':
        return dict(bytes=4.0 * n * P + 16.0 * px, flops=ev * fwd)
    if kind == 'raster':
        return dict(bytes=8.0 * n * P + 32.0 * px, flops=ev * (fwd + bwd))
    if kind == 'grow':
        # parameters and moments copied; per view two images and the counts
        return dict(bytes=24.0 * n * P + GROW_VIEWS * (4.0 * n * P + 12.0 * px),
                    flops=GROW_VIEWS * ev * 2 * fwd)
    # a training step: parameters and both moments read and written, the target read
    return dict(bytes=24.0 * n * P + (16.0 if kind == 'fit' else 12.0) * px,
                flops=ev * (fwd + bwd))


# -- 64-bit values ------------------------------------------------------------

def exact(case, seed):
    kind = case['kind']
    if kind == 'photo':
        return _exact_photo(prepare(case, seed))
    if kind == 'decode':
        return _exact_decode(prepare(case, seed))
    if kind == 'raster':
        px = case['w'] * case['h']
        if px <= 512 * 512 and case['n'] <= 50_000:
            return _exact_raster(prepare(case, seed))
    return None


def _exact_photo(s):
    x = s['img'].double().requires_grad_(True)
    y = s['tgt'].double()
    _, h, w = x.shape
    k = torch.exp(-(torch.arange(11, dtype=torch.float64) - 5.0) ** 2 / (2 * 1.5 ** 2))
    k = (k / k.sum()).tolist()

    def window(v):
        p = torch.nn.functional.pad(v, (5, 5))
        v = sum(k[t] * p[..., t:t + w] for t in range(11))
        p = torch.nn.functional.pad(v, (0, 0, 5, 5))
        return sum(k[t] * p[..., t:t + h, :] for t in range(11))

    mx, my = window(x), window(y)
    vx, vy, cxy = window(x * x) - mx * mx, window(y * y) - my * my, window(x * y) - mx * my
    c1, c2 = 0.01 ** 2, 0.03 ** 2
    ssim = ((2 * mx * my + c1) * (2 * cxy + c2) / ((mx * mx + my * my + c1) * (vx + vy + c2))).mean()
    l1 = (x - y).abs().mean()
    e = 0.8 * l1 + 0.2 * (1.0 - ssim)
    e.backward()
    return dict(loss=torch.stack([e, l1, ssim]).detach(), dI=x.grad)


def _rounded(x, kind):
    """x rounded to a narrower type, with the gradient of x itself."""
    r = x.detach().float() if kind == 'f32' else x.detach().float().bfloat16()
    return x + (r.double() - x.detach())


def _exact_decode(s):
    a = {k: v.double().requires_grad_(k != 'pos') for k, v in s['a'].items()}
    m = {k: v.double().requires_grad_(True) for k, v in s['m'].items()}
    A = a['feat'].shape[1]
    R = torch.tensor(list(s['cam'].R), dtype=torch.float64, device='cuda').view(3, 3)
    t = torch.tensor(list(s['cam'].t), dtype=torch.float64, device='cuda')
    d = (-R.T @ t)[:, None] - a['pos']
    x = _rounded(torch.cat([a['feat'], d / d.norm(dim=0, keepdim=True)]), 'bf16')
    h = _rounded(torch.relu(_rounded(m['w1'], 'bf16') @ x + m['b1'][:, None]), 'bf16')
    w2, rows = _rounded(m['w2'], 'bf16'), (0, 10, 40, 110)
    y = torch.cat([w2[rows[i]:rows[i + 1]] @ h[32 * i:32 * i + 32] for i in range(3)])
    y = y + m['b2'][:, None]
    col, cov = y[10:40].view(10, 3, A), y[40:].view(10, 7, A)
    off = a['offsets'].view(10, 3, A)
    q = cov[:, 3:]
    ch = dict(means=a['pos'] + off * a['scaling'][:3],
              log_scales=a['scaling'][3:] * torch.sigmoid(cov[:, :3]),
              quats=q / q.norm(dim=1, keepdim=True),
              opacity_logits=torch.relu(torch.tanh(y[:10])), sh=torch.sigmoid(col))
    # child j of anchor i is Gaussian j A + i
    ch = {k: (v.reshape(-1) if v.dim() == 2 else v.transpose(0, 1).reshape(v.shape[1], 10 * A))
          for k, v in ch.items()}
    sum((ch[k] * s['dchild'][k].double()).sum() for k in ch).backward()
    return dict(children={k: v.detach() for k, v in ch.items()},
                danchors={k: a[k].grad for k in ('feat', 'offsets', 'scaling')},
                dmlp={k: m[k].grad for k in MLP_NAMES})


def _sh_basis(deg, d):
    x, y, z = d
    one = torch.ones_like(x)
    pi = math.pi
    Y = [one * (0.5 / math.sqrt(pi))]
    if deg >= 1:
        k = math.sqrt(3 / (4 * pi))
        Y += [-k * y, k * z, -k * x]
    if deg >= 2:
        k = math.sqrt(15 / pi)
        Y += [0.5 * k * x * y, -0.5 * k * y * z,
              0.25 * math.sqrt(5 / pi) * (2 * z * z - x * x - y * y),
              -0.5 * k * x * z, 0.25 * k * (x * x - y * y)]
    if deg >= 3:
        ka, kc = 0.25 * math.sqrt(35 / (2 * pi)), 0.25 * math.sqrt(21 / (2 * pi))
        kb = math.sqrt(105 / pi)
        Y += [-ka * y * (3 * x * x - y * y), 0.5 * kb * x * y * z,
              -kc * y * (4 * z * z - x * x - y * y),
              0.25 * math.sqrt(7 / pi) * z * (2 * z * z - 3 * x * x - 3 * y * y),
              -kc * x * (4 * z * z - x * x - y * y), 0.25 * kb * z * (x * x - y * y),
              -ka * x * (x * x - 3 * y * y)]
    return torch.stack(Y)


def _exact_records(p, deg, cam):
    """Splat records [11, n] (u, v, a, b, c, t, o, depth channel, r, g, b) as they are stored (32
    bits), the depth that orders them, and which Gaussians are in front of the camera."""
    R = torch.tensor(cam.R, dtype=torch.float64, device='cuda')
    t = torch.tensor(cam.t, dtype=torch.float64, device='cuda')
    q = p['quats'] / p['quats'].norm(dim=0, keepdim=True)
    w, x, y, z = q
    rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]).view(3, 3, -1)
    M = rot * torch.exp(p['log_scales'])[None]
    pc = R @ p['means'] + t[:, None]
    front = pc[2] > cam.near
    pz = torch.where(front, pc[2], torch.ones_like(pc[2]))
    xr, yr = pc[0] / pz, pc[1] / pz
    lx, ly = 1.3 * cam.width / (2 * cam.fx), 1.3 * cam.height / (2 * cam.fy)
    J0 = (cam.fx / pz)[None] * R[0][:, None] - (cam.fx * xr.clamp(-lx, lx) / pz)[None] * R[2][:, None]
    J1 = (cam.fy / pz)[None] * R[1][:, None] - (cam.fy * yr.clamp(-ly, ly) / pz)[None] * R[2][:, None]
    m0, m1 = (J0[:, None] * M).sum(0), (J1[:, None] * M).sum(0)
    A, B, C = (m0 * m0).sum(0) + 0.3, (m0 * m1).sum(0), (m1 * m1).sum(0) + 0.3
    det = A * C - B * B
    o = torch.sigmoid(p['opacity_logits'])
    eye = -(R.T @ t)
    d = p['means'] - eye[:, None]
    Y = _sh_basis(deg, d / d.norm(dim=0, keepdim=True))
    rgb = torch.relu((p['sh'] * Y[:, None]).sum(0) + 0.5)
    chan = 1.0 / pz if cam.depth_mode else pz
    rec = torch.stack([cam.fx * xr + cam.cx, cam.fy * yr + cam.cy, C / det, -B / det, A / det,
                       2.0 * torch.log(255.0 * o), o, chan, rgb[0], rgb[1], rgb[2]])
    return _rounded(rec, 'f32'), pz.detach().float(), front & (det > 0)


def _exact_raster(s):
    case, cam = s['case'], s['cam']
    p = {k: v.double().requires_grad_(True) for k, v in s['p'].items()}
    full, z, front = _exact_records(p, case['deg'], cam)
    rec = full.detach().requires_grad_(True)
    u, v, a, b, c, t = rec.detach()[:6]
    det = a * c - b * b
    ok = front & (t > 0) & (det > 0)
    hx, hy = torch.sqrt((t * c / det).clamp_min(0)), torch.sqrt((t * a / det).clamp_min(0))
    order = torch.sort(z, stable=True).indices
    order = order[ok[order]]
    h, w = case['h'], case['w']
    image = torch.zeros(3, h, w, dtype=torch.float64, device='cuda')
    depth = torch.zeros(h, w, dtype=torch.float64, device='cuda')
    amax, stop = float(torch.tensor(0.99)), float(torch.tensor(1e-4))
    dD = s['dD'].double() if s['dD'] is not None else None
    for y0 in range(0, h, 16):
        for x0 in range(0, w, 16):
            ny, nx = min(16, h - y0), min(16, w - x0)
            near = ((u + hx >= x0) & (u - hx <= x0 + nx) & (v + hy >= y0) & (v - hy <= y0 + ny))
            pick = order[near[order]]
            if not len(pick):
                continue
            r = rec[:, pick]
            py, px = torch.meshgrid(torch.arange(ny, device='cuda') + y0 + 0.5,
                                    torch.arange(nx, device='cuda') + x0 + 0.5, indexing='ij')
            dx = px.reshape(-1, 1).double() - r[0]
            dy = py.reshape(-1, 1).double() - r[1]
            Q = dx * (r[2] * dx + 2 * r[3] * dy) + r[4] * dy * dy
            al = torch.where(Q > r[5], torch.zeros_like(Q),
                             (r[6] * torch.exp(-0.5 * Q)).clamp(max=amax))
            live = torch.cumprod(1 - al.detach(), 1) >= stop
            al = al * live
            T = torch.cumprod(1 - al, 1)
            wgt = al * torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], 1)
            col, dep = wgt @ r[8:11].T, wgt @ r[7]      # the background is black
            sl = (slice(y0, y0 + ny), slice(x0, x0 + nx))
            dI = s['dI'][(slice(None),) + sl].double().reshape(3, -1)
            loss = (col.T * dI).sum()
            if dD is not None:
                loss = loss + (dep * dD[sl].reshape(-1)).sum()
            loss.backward()
            image[(slice(None),) + sl] = col.detach().T.reshape(3, ny, nx)
            depth[sl] = dep.detach().reshape(ny, nx)
    torch.autograd.backward(full, rec.grad if rec.grad is not None else torch.zeros_like(rec))
    return dict(image=image, depth=depth, grads={k: p[k].grad for k in p})
