# minimax-like fits (Chebyshev interpolation in long double) of
#   P(z): atanh(s)/s = 1 + z P(z), z = s^2 <= ((sqrt2-1)/(sqrt2+1))^2
#   A(z): atan(r)/r  = 1 + z A(z), z = r^2 <= tan(pi/16)^2
import numpy as np
L=np.longdouble
def series(z,sign,n=60):
    t=L(0)
    for k in range(n,-1,-1): t = t*(sign*z) + L(1)/L(2*k+3)
    return t*(L(sign))
def fit(zmax,deg,sign):
    # Remez-free: Chebyshev nodes interpolation of sum, monomials in z
    n=deg+1
    x=np.cos((2*np.arange(n)+1)*np.pi/(2*n)).astype(L)
    z=(x+1)/2*L(zmax)
    f=np.array([series(zz,sign) for zz in z],dtype=L)
    # Newton divided differences -> monomial
    c=f.copy()
    for j in range(1,n):
        for i in range(n-1,j-1,-1): c[i]=(c[i]-c[i-1])/(z[i]-z[i-j])
    p=np.zeros(n,dtype=L); p[0]=c[n-1]
    deg_=0
    for i in range(n-2,-1,-1):
        q=np.zeros(n,dtype=L); q[1:deg_+2]=p[:deg_+1]; q[:deg_+1]-=z[i]*p[:deg_+1]; q[0]+=c[i]; p=q; deg_+=1
    d=p.astype(np.float64)
    zz=np.linspace(0,float(zmax),20001).astype(L)
    ref=series(zz,sign); v=L(0)
    for k in range(n-1,-1,-1): v=v*zz+L(d[k])
    print("deg",deg,"err rel to 1: %.2e"%float(np.max(np.abs((v-ref)*zz))))
    return d
zl=((2**.5-1)/(2**.5+1))**2*1.0005; za=np.tan(np.pi/16)**2*1.0005
for deg in (7,8): 
    print([float.hex(v) for v in fit(zl,deg,1)]); print([repr(float(v)) for v in fit(zl,deg,1)])
for deg in (8,9):
    print([repr(float(v)) for v in fit(za,deg,-1)])
