// The stand-ins of stubs.cpp, with requests that ask for graphs and a set-up
// that refuses them (test infrastructure).
#define poisson_setup stub_setup
#define poisson_default_opts stub_default_opts
#include "stubs.cpp"
#undef poisson_setup
#undef poisson_default_opts
extern "C" int32_t poisson_setup(const ibm_grid *g, const uint8_t *flags, const ibm_stencils *st, const poisson_opts *o,
                                 size_t *bytes, poisson_ctx **out)
{
    return o->use_graph ? IBM_EINVAL : stub_setup(g, flags, st, o, bytes, out);
}
extern "C" void poisson_default_opts(poisson_opts *o)
{
    stub_default_opts(o);
    o->use_graph = 1;
}
